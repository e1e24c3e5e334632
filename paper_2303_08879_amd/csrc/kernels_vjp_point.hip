// Reverse level kernels of plans with every mode detected (Algorithm 1), one
// launch per level (the work of a tile is in vjp_point_units.h).
#include <algorithm>

#include "vjp_point_units.h"

namespace fd {

// Two wavefronts per SIMD asked for: the compiler then keeps the MFMA operands
// and results out of the accumulation registers (8 modes, b = 0: 200 -> 184).
template <int MD, bool ODD, int T, typename R>
__global__ __launch_bounds__(kThreads, 2) void k_vjp_point(DevPlan P, VjpPtrs<R> V, const uint64_t* __restrict__ mt,
                                                        const cx<R>* __restrict__ Ai, const cx<R>* __restrict__ bi,
                                                        int S, int nwork, int nwide, int wide_off,
                                                        double2* __restrict__ partial) {
  constexpr int NP = 2 * MD, NR = NP + 1, NPAIR = NP * NR, SL = 16 * T;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  R* sq = reinterpret_cast<R*>(smem_raw);
  uint64_t* hp = reinterpret_cast<uint64_t*>(sq + 2 * (kMaxCut + 4));
  uint64_t* gp = hp + pt_table_entries(MD);
  uint64_t* xp = gp + pt_table_entries(MD);
  cx<R>* turn = reinterpret_cast<cx<R>*>(hp + pt_vjp_entries(MD));
  int* rows = reinterpret_cast<int*>(turn + (kThreads / 64) * kPtPos * kTurn);
  int* spn = rows + (kThreads / 64) * pt_row_ints(MD, T);
  const int wave = threadIdx.x >> 6;
  turn += wave * kPtPos * kTurn;
  rows += wave * pt_row_ints(MD, T);
  pt_load_tables<R>(P, MD, sq, spn);
  pt_fill_vjp_pointers<MD, ODD, R>(V, hp, gp, xp);
  VjpPtConst<MD, ODD, R> C;
  C.load(P, Ai, bi);
  __syncthreads();
  const VjpPtLevel<R> L{hp, gp, xp, sq, sq + (kMaxCut + 4), spn, V.fcur[0], V.d0cur, V.gcur[0], V.gf0nxt != nullptr};
  VjpPtSums<MD, R> Z;
  Z.zero();
  if (T == 1 && (int)blockIdx.x < nwide) {
    // the first tiles, which take several bridges: one workgroup each
    cx<R>* shared = reinterpret_cast<cx<R>*>(reinterpret_cast<unsigned char*>(smem_raw) + wide_off);
    vjp_point_tile<MD, ODD, 1, R, true>(P, L, C, Z, mt, S, 16 * (int)blockIdx.x, nwork, turn, rows, shared, wave);
  } else {
    const int stride = (gridDim.x - nwide) * (kThreads / 64) * SL;
    for (int base = 16 * nwide + ((blockIdx.x - nwide) * (kThreads / 64) + wave) * SL; base < nwork; base += stride)
      vjp_point_tile<MD, ODD, T, R>(P, L, C, Z, mt, S, base, nwork, turn, rows);
  }
  // fold the wavefronts' pair tables (fixed order) into this workgroup's slot
  cx<double>* red = reinterpret_cast<cx<double>*>(smem_raw);
  __syncthreads();
  Z.template store<ODD>(red + (size_t)wave * NPAIR);
  __syncthreads();
  double2* slot = partial + (size_t)blockIdx.x * NPAIR;
  for (int p = threadIdx.x; p < NPAIR; p += blockDim.x) {
    if (!ODD && p % NR == NP) continue;   // the bbar column without odd levels: zero
    double sx = 0.0, sy = 0.0;
    for (int wv = 0; wv < kThreads / 64; ++wv) {
      sx += red[(size_t)wv * NPAIR + p].x;
      sy += red[(size_t)wv * NPAIR + p].y;
    }
    const double2 v = slot[p];
    slot[p] = make_double2(v.x + sx, v.y + sy);
  }
}

// Tiles of a level that get a workgroup of their own (those whose points take
// more than one bridge), while the level leaves the device idle wavefronts.
static int wide_tiles(const Plan& Pl, int S) {
  if (Pl.MD < 2 || Pl.ncnt[S] > 16 * kWideTiles) return 0;
  return (int)((Pl.ncnt[(size_t)(Pl.smax + 1) + S] + 15) / 16);
}
int vjp_point_grid(const Plan& Pl, int S) {
  const int nwork = (int)Pl.ncnt[S], wide = wide_tiles(Pl, S);
  const int per = kThreads / 64 * 16 * (nwork >= kPointTileMin ? 4 : 1);
  return std::min(wide + (std::max(nwork - 16 * wide, 0) + per - 1) / per, kPartialSlots - 1);
}

template <int T, typename R>
static hipError_t launch_t(const Plan& Pl, const DevPlan& P, bool odd, int S, const VjpPtrs<R>& V, const cx<R>* A,
                           const cx<R>* b, int nwork, double2* partial, hipStream_t st) {
  // (the rows shared by a workgroup's tile after everything else)
  const size_t wide_off = (pt_lds_bytes(Pl, T, kThreads / 64, 3) + kPtPos * 8 +
                           (size_t)(kThreads / 64) * kPtPos * kTurn * sizeof(cx<R>) + 15) / 16 * 16;
  const int nwide = T == 1 ? wide_tiles(Pl, S) : 0;
  const size_t shm =
      std::max(wide_off + (nwide ? (size_t)wide_entries(Pl.MD) * sizeof(cx<R>) : 0),
               (size_t)(kThreads / 64) * 2 * Pl.MD * (2 * Pl.MD + 1) * sizeof(cx<double>));
  const uint64_t* mt = Pl.d_mtab ? Pl.d_mtab + Pl.lvl[S] : nullptr;
  const int grid = vjp_point_grid(Pl, S);
#define FD_VJP_POINT(MDV)                                                                                          \
  case MDV:                                                                                                        \
    if (odd)                                                                                                       \
      hipLaunchKernelGGL((k_vjp_point<MDV, true, T, R>), dim3(grid), dim3(kThreads), shm, st, P, V, mt, A, b, S,   \
                         nwork, nwide, (int)wide_off, partial);                                                                        \
    else                                                                                                           \
      hipLaunchKernelGGL((k_vjp_point<MDV, false, T, R>), dim3(grid), dim3(kThreads), shm, st, P, V, mt, A, b, S,  \
                         nwork, nwide, (int)wide_off, partial);                                                                        \
    break;
  switch (Pl.MD) {
    FD_VJP_POINT(1)
    FD_VJP_POINT(2)
    FD_VJP_POINT(3)
    FD_VJP_POINT(4)
    FD_VJP_POINT(5)
    FD_VJP_POINT(6)
    FD_VJP_POINT(7)
    FD_VJP_POINT(8)
    default:
      return hipErrorInvalidValue;
  }
#undef FD_VJP_POINT
  return hipGetLastError();
}

template <typename R>
hipError_t launch_vjp_point_level(const Plan& Pl, const DevPlan& P, bool odd, int S, const VjpPtrs<R>& V,
                                  const cx<R>* A, const cx<R>* b, int nwork, double2* partial, hipStream_t st) {
  return nwork >= kPointTileMin ? launch_t<4, R>(Pl, P, odd, S, V, A, b, nwork, partial, st)
                                : launch_t<1, R>(Pl, P, odd, S, V, A, b, nwork, partial, st);
}
template hipError_t launch_vjp_point_level<float>(const Plan&, const DevPlan&, bool, int, const VjpPtrs<float>&,
                                                  const cx<float>*, const cx<float>*, int, double2*, hipStream_t);
template hipError_t launch_vjp_point_level<double>(const Plan&, const DevPlan&, bool, int, const VjpPtrs<double>&,
                                                   const cx<double>*, const cx<double>*, int, double2*, hipStream_t);

}  // namespace fd
