// Forward level kernels of plans with every mode detected (Algorithm 1), values
// or values and tangents (forward mode, DUAL): one launch per sweep step, the
// points of the level in tiles of 16 columns on the matrix cores (pt_units.h).
#include <algorithm>

#include "pt_units.h"

namespace fd {

template <int MD, bool ODD, bool DUAL, typename R>
__global__ __launch_bounds__(kThreads, 2) void k_fwd_point(DevPlan P, LevelPtrs<R> L, const uint64_t* __restrict__ mt,
                                                           const cx<R>* __restrict__ Ai, const cx<R>* __restrict__ bi,
                                                           int S, PtItems I, int64_t dT) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  R* sq = reinterpret_cast<R*>(smem_raw);
  uint64_t* rd = reinterpret_cast<uint64_t*>(sq + 2 * (kMaxCut + 4));
  uint64_t* wr = rd + pt_table_entries(MD);
  int* rows = reinterpret_cast<int*>(wr + pt_table_entries(MD));
  int* spn = rows + (kThreads / 64) * pt_row_ints(MD, 1);
  rows += (threadIdx.x >> 6) * pt_row_ints(MD, 1);
  pt_load_tables<R>(P, MD, sq, spn);
  pt_fill_pointers<MD, ODD, R>(L, rd, wr);
  PtConst<MD, ODD, DUAL, R> C;
  C.load(P, Ai, bi, dT);
  __syncthreads();
  const PtLds<R> Y{sq, sq + (kMaxCut + 4), spn, rd, wr};
  int K = 0, base = 0, n = 0;
  if (!pt_item<MD>(I, blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), &K, &base, &n))
    return;
  fwd_point_item<MD, ODD, DUAL, R>(P, Y, C, L.f0cur, L.f0nxt != nullptr, mt, S, K, base, n, rows, dT);
}

// Digits of every lattice point in node order (8 bits per mode, mode j at bit
// 8 j), one thread per point; run once when the plan's tables are made. Built by
// the host the table of 735 thousand points (8 modes, at most 16 photons) made
// the plan's first call take 6065 us, built here 450; with it the 8-mode cutoff 8
// step (16.8 million points) takes 6717 us, unranking each point in each level
// kernel 7110.
template <int MD>
__global__ __launch_bounds__(kThreads) void k_digit_table(DevPlan P, int64_t n, uint64_t* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  int* spn = reinterpret_cast<int*>(smem_raw);
  for (int i = threadIdx.x; i < (MD + 1) * P.pnw; i += blockDim.x) spn[i] = P.pn[i];
  __syncthreads();
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
    int lo = 0, hi = P.smax;   // the level: the last one that starts at or before t
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (P.lvl[mid] <= t)
        lo = mid;
      else
        hi = mid - 1;
    }
    int m[MD], s[MD + 1];
    unrank<MD>(spn, P.pnw, P.CD, lo, (int)(t - P.lvl[lo]), m, s);
    uint64_t pk = 0;
#pragma unroll
    for (int d = 0; d < MD; ++d) pk |= (uint64_t)m[d] << (8 * d);
    out[t] = pk;
  }
}

hipError_t fill_digit_table(const Plan& Pl) {
  const DevPlan P = make_devplan(Pl, true);
  const int64_t n = Pl.nodes_total;
  const unsigned grid = (unsigned)std::min<int64_t>((n + kThreads - 1) / kThreads, 8192);
  const size_t shm = (size_t)(Pl.MD + 1) * (Pl.smax + 3) * sizeof(int);
#define FD_DIGITS(MDV)                                                                                       \
  case MDV:                                                                                                  \
    hipLaunchKernelGGL((k_digit_table<MDV>), dim3(grid), dim3(kThreads), shm, nullptr, P, n, Pl.d_mtab);     \
    break;
  switch (Pl.MD) {
    FD_DIGITS(1)
    FD_DIGITS(2)
    FD_DIGITS(3)
    FD_DIGITS(4)
    FD_DIGITS(5)
    FD_DIGITS(6)
    FD_DIGITS(7)
    FD_DIGITS(8)
    default:
      return hipErrorInvalidValue;
  }
#undef FD_DIGITS
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : hipStreamSynchronize(nullptr);
}

template <typename R>
hipError_t launch_fwd_point_level(const Plan& Pl, const DevPlan& P, bool odd, int S, const LevelPtrs<R>& L,
                                  const cx<R>* A, const cx<R>* b, hipStream_t st, int64_t dT) {
  const PtItems I = pt_items(Pl, S);
  int units = 0;
  for (int K = 0; K < Pl.MD; ++K) units += I.tiles(K);
  const int grid = (units + kThreads / 64 - 1) / (kThreads / 64);
  const size_t shm = pt_lds_bytes(Pl, 1, kThreads / 64, 2);
  const uint64_t* mt = Pl.d_mtab ? Pl.d_mtab + Pl.lvl[S] : nullptr;
#define FD_LAUNCH(MDV, ODD, DUAL)                                                                                  \
  hipLaunchKernelGGL((k_fwd_point<MDV, ODD, DUAL, R>), dim3(grid), dim3(kThreads), shm, st, P, L, mt, A, b, S, I,  \
                     dT)
#define FD_LAUNCH_POINT(MDV)           \
  case MDV:                            \
    if (dT)                            \
      FD_LAUNCH(MDV, true, true);      \
    else if (odd)                      \
      FD_LAUNCH(MDV, true, false);     \
    else                               \
      FD_LAUNCH(MDV, false, false);    \
    break;
  switch (Pl.MD) {
    FD_LAUNCH_POINT(1)
    FD_LAUNCH_POINT(2)
    FD_LAUNCH_POINT(3)
    FD_LAUNCH_POINT(4)
    FD_LAUNCH_POINT(5)
    FD_LAUNCH_POINT(6)
    FD_LAUNCH_POINT(7)
    FD_LAUNCH_POINT(8)
    default:
      return hipErrorInvalidValue;
  }
#undef FD_LAUNCH_POINT
#undef FD_LAUNCH
  return hipGetLastError();
}
template hipError_t launch_fwd_point_level<float>(const Plan&, const DevPlan&, bool, int, const LevelPtrs<float>&,
                                                  const cx<float>*, const cx<float>*, hipStream_t, int64_t);
template hipError_t launch_fwd_point_level<double>(const Plan&, const DevPlan&, bool, int, const LevelPtrs<double>&,
                                                   const cx<double>*, const cx<double>*, hipStream_t, int64_t);

}  // namespace fd
