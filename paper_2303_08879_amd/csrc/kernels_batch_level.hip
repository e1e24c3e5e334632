// Level kernels of the batched forward: one step of every circuit of a class.
#include "batch_level.h"
#include "pt_units.h"

namespace fd {

template <int MD, bool ODD, typename R>
__global__ __launch_bounds__(kThreads, 2) void k_batch_point(const BatchCirc<R>* __restrict__ circs,
                                                          const BatchItem* __restrict__ items, int S) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const BatchItem I = items[blockIdx.x];
  const BatchCirc<R>* __restrict__ C = circs + I.circ;
  R* sq = reinterpret_cast<R*>(smem_raw);
  uint64_t* rd = reinterpret_cast<uint64_t*>(sq + 2 * (kMaxCut + 4));
  uint64_t* wr = rd + pt_table_entries(MD);
  int* rows = reinterpret_cast<int*>(wr + pt_table_entries(MD));
  int* spn = rows + (kThreads / 64) * pt_row_ints(MD, 1);
  rows += (threadIdx.x >> 6) * pt_row_ints(MD, 1);
  const DevPlan& P = C->P;
  const R* sqt = static_cast<const R*>(load_global(&P.sqt));
  const int* pn = load_global(&P.pn);
  for (int i = threadIdx.x; i < 2 * (kMaxCut + 4); i += blockDim.x) sq[i] = sqt[i];
  for (int i = threadIdx.x; i < (MD + 1) * P.pnw; i += blockDim.x) spn[i] = pn[i];
  const BatchLevel<R> L = batch_level(C, S);
  pt_fill_pointers<MD, ODD, R>(L, rd, wr);
  const cx<R>* Ai = load_global(&C->Ai);
  PtConst<MD, ODD, false, R> Q;
  Q.load(P, Ai, Ai + 4 * MD * MD, 0);
  __syncthreads();
  const PtLds<R> Y{sq, sq + (kMaxCut + 4), spn, rd, wr};
  const uint64_t* mt = load_global(&C->mtab);
  const int64_t* lvl = load_global(&P.lvl);
  if (mt) mt += lvl[S];
  PtItems N;
#pragma unroll
  for (int K = 0; K < MD; ++K) N.n[K] = (int)(lvl[K * (P.smax + 2) + S + 1] - lvl[K * (P.smax + 2) + S]);
  for (int u = I.u0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); u < I.u1; u += kThreads / 64) {
    int K = 0, base = 0, n = 0;
    if (!pt_item<MD>(N, u, &K, &base, &n)) break;
    fwd_point_item<MD, ODD, false, R>(P, Y, Q, L.f0cur, L.f0nxt != nullptr, mt, S, K, base, n, rows);
  }
}

template <int MD, int NQ, typename R>
__global__ __launch_bounds__(kBT * kFwdWaves) void k_batch_block(const BatchCirc<R>* __restrict__ circs,
                                                                 const BatchItem* __restrict__ items, int S) {
  constexpr int NPOS = NQ + 2 * MD;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const BatchItem I = items[blockIdx.x];
  const BatchCirc<R>* __restrict__ C = circs + I.circ;
  ChunkGeo G;
  G.C0 = C->P.udims[0];
  G.R0 = C->P.ustride[0];
  G.RC = I.RC;
  G.nchunks = I.nchunks;
  cx<R>* lf0 = reinterpret_cast<cx<R>*>(smem_raw);          // (RC + 2) rows
  cx<R>* lpk = lf0 + (size_t)(G.RC + 2) * G.R0;             // MD x (RC + 1) rows
  cx<R>* sA = lpk + (size_t)MD * (G.RC + 1) * G.R0;         // A (NPOS x NPOS) then b (NPOS)
  R* sq = reinterpret_cast<R*>(sA + NPOS * NPOS + NPOS);
  R* isq = sq + (kMaxCut + 4);
  for (int v = threadIdx.x; v < kMaxCut + 4; v += blockDim.x) {
    sq[v] = sqrt(R(v));
    isq[v] = v ? R(1) / sqrt(R(v)) : R(0);
  }
  const cx<R>* Ai = load_global(&C->Ai);
  for (int i = threadIdx.x; i < NPOS * NPOS + NPOS; i += blockDim.x) sA[i] = ld(Ai + i);
  const BatchLevel<R> L = batch_level(C, S);
  // the unit's first barrier orders these LDS writes before their reads
  for (int u = I.u0; u < I.u1; ++u) {
    const int r = u / G.nchunks, c = u - r * G.nchunks;
    fwd_block_unit<MD, NQ, R, BatchLevel<R>, cx<R>, false, kFwdWaves>(C->P, L, sA, sA + NPOS * NPOS, sq, isq, S, r,
                                                                      c, G, lf0, lpk);
    __syncthreads();   // the next unit overwrites the rows
  }
}

template <typename R>
hipError_t launch_batch_level(const BatchLaunch& a, hipStream_t st) {
  const BatchCirc<R>* circs = static_cast<const BatchCirc<R>*>(a.circs);
#define FD_LAUNCH(KERN, THREADS)                                                                            \
  {                                                                                                         \
    if (a.shm > 65536)                                                                                      \
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&KERN),                                       \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.shm);                    \
    hipLaunchKernelGGL(KERN, dim3((unsigned)a.nitems), dim3(THREADS), a.shm, st, circs, a.items, a.S);      \
  }
#define FD_CASE(MDV)                                                   \
  case MDV:                                                            \
    if (a.kind == 0) {                                                 \
      if (a.odd)                                                       \
        FD_LAUNCH((k_batch_point<MDV, true, R>), kThreads)             \
      else                                                             \
        FD_LAUNCH((k_batch_point<MDV, false, R>), kThreads)            \
    } else if (a.nq == 2) {                                            \
      FD_LAUNCH((k_batch_block<MDV, 2, R>), kBT* kFwdWaves)            \
    } else {                                                           \
      FD_LAUNCH((k_batch_block<MDV, 4, R>), kBT* kFwdWaves)            \
    }                                                                  \
    break;
  switch (a.MD) {
    FD_CASE(1)
    FD_CASE(2)
    FD_CASE(3)
    FD_CASE(4)
    FD_CASE(5)
    FD_CASE(6)
    FD_CASE(7)
    FD_CASE(8)
    default:
      return hipErrorInvalidValue;
  }
#undef FD_CASE
#undef FD_LAUNCH
  return hipGetLastError();
}

template hipError_t launch_batch_level<float>(const BatchLaunch&, hipStream_t);
template hipError_t launch_batch_level<double>(const BatchLaunch&, hipStream_t);

}  // namespace fd
