// fill.hip -- the fill of one plan (Sec. 3.2 with the relations of Sec. 4.1 /
// 5.1) without a launch or a barrier per level: 2D plans that fit in LDS by
// one workgroup per field (fill_lds2), other plans without coupled units by
// every ghost waiting for its own corners across the chip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "gcr_fill.hpp"

namespace gcr {

__global__ __launch_bounds__(1024) void k_fill_lds(FillArgs A, const int32_t* __restrict__ lev_off,
                                                   int nlev) {
  extern __shared__ double s_lds[];
  const int f = blockIdx.x;
  fill_lds2(A.P, lev_off, nlev, A.f[f], A.b[f], A.bt[f], A.kind[f], s_lds);
}

bool fill_lds_fits(const PlanD& P) {
  return fill_lds_ok(P) && fill_lds_bytes(P.ng, P.nunits) <= 160 * 1024;
}

// Few ghosts take a workgroup of four waves, others sixteen (their gathers
// are the wait).
gcr_status launch_fill_lds(const FillArgs& A, const int32_t* d_lev_off, int nlev,
                           hipStream_t st) {
  static std::mutex mu;
  static bool ready = false;
  const size_t lds = fill_lds_bytes(A.P.ng, A.P.nunits);
  if (lds > 65536) {
    std::lock_guard<std::mutex> lk(mu);
    if (!ready && hipFuncSetAttribute(reinterpret_cast<const void*>(&k_fill_lds),
                                      hipFuncAttributeMaxDynamicSharedMemorySize,
                                      160 * 1024) != hipSuccess)
      return GCR_E_HIP;
    ready = true;
  }
  k_fill_lds<<<A.nf, A.P.ng <= 512 ? 256 : 1024, lds, st>>>(A, d_lev_off, nlev);
  return hipGetLastError() == hipSuccess ? GCR_OK : GCR_E_HIP;
}

// --------------------------------------------------------------------------
// Fill by waiting.  k_fill_open computes level 1, which reads fluid cells
// only, and stores kFillOpen into every other ghost slot.  k_fill_flow then
// has one thread per ghost of the other levels and field: it gathers its
// fluid corners and weights, and polls the slots of its ghost corners (the
// code's mask says which they are) until each holds a value, at agent scope:
// the value is the flag, so nothing else is shared and nothing is kept from
// one call for another.  A level costs one store-to-load trip across the
// chip, about 0.5 us, where a launch per level cost 6.5 us.
//
// A ghost reads lower levels only, so workgroups wait for earlier ones
// (canonical order is by level; fields one after another); the hardware
// starts workgroups in order, so the one the others wait for runs.  That is
// not promised, so a wait is bounded (`polls`): a thread that passes it
// computes the ghosts it waits for itself (fill_help), and the fill ends
// whichever workgroups run.
// Bound by the chain of levels.  256^3 sphere, 18,500 ghosts, 11 levels, four
// fields: 23.5 us for the two launches against 87 for eleven (25 with a third to
// sweep again after a wait that gave up).
// --------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void k_fill_open(FillArgs A, int n1) {
  const int p = blockIdx.x * 256 + threadIdx.x, f = blockIdx.y;
  if (p >= A.P.ng) return;
  if (p < n1) fill_single<D, true>(A.P, p, A.f[f], A.b[f], A.bt[f], A.kind[f]);
  else A.f[f][A.P.cell[p]] = __longlong_as_double((long long)kFillOpen);
}

template <int D>
__global__ __launch_bounds__(256) void k_fill_flow(FillArgs A, int n1, int polls) {
  const int f = blockIdx.y;
  const int p = min(n1 + (int)(blockIdx.x * 256 + threadIdx.x), A.P.ng - 1);   // (the last: again)
  fill_wait<D>(A.P, p, A.f[f], A.b[f], A.bt[f], A.kind[f], polls);
}

template <int D>
static void fill_flow(const FillArgs& A, int n1, int polls, hipStream_t st) {
  const unsigned nf = (unsigned)A.nf;
  k_fill_open<D><<<dim3((unsigned)((A.P.ng + 255) / 256), nf), 256, 0, st>>>(A, n1);
  if (A.P.ng <= n1) return;
  k_fill_flow<D><<<dim3((unsigned)((A.P.ng - n1 + 255) / 256), nf), 256, 0, st>>>(A, n1, polls);
}

// n1: ghosts of level 1; polls: of a wait before the thread helps itself
gcr_status launch_fill_flow(const FillArgs& A, int n1, int polls, hipStream_t st) {
  if (A.P.g.dim == 2) fill_flow<2>(A, n1, polls, st);
  else fill_flow<3>(A, n1, polls, st);
  return hipGetLastError() == hipSuccess ? GCR_OK : GCR_E_HIP;
}

}  // namespace gcr
