// Forward block kernel (Algorithm 2) and its per-level launches, compiled in
// eight translation units.
#pragma once

#include <algorithm>

#include "fwd_units.h"

namespace fd {

// Algorithm 2: one workgroup of WV wavefronts per (lattice point, chunk of
// undetected rows).  Chunks of about 112 entries per wavefront over four
// wavefronts leave fewer rows to the halo than one-wavefront chunks (the
// 5-mode conditional forward sweep 2.29 -> 1.78 ms, the 4-mode one 0.45 ->
// 0.40 ms, the 6-mode gradient circuit 4.61 -> 3.75 ms).
// E = dual<R> carries every amplitude's tangent along (forward mode), dT
// bytes after the value.  ST: the rows stream from HBM (blocks whose rows do
// not fit the LDS); the bridge pivot blocks then go to the workgroup's slot
// of `slots` (slot_len entries each).
template <int MD, int NQ, typename R, typename E, bool ST, int WV>
__global__ __launch_bounds__(kBT * WV) void k_fwd_block(DevPlan P, LevelPtrs<R> L, const cx<R>* __restrict__ Ai,
                                                   const cx<R>* __restrict__ bi, int S, int nwork, ChunkGeo G,
                                                   int64_t dT, cx<R>* slots, int64_t slot_len) {
  static_assert(!ST || std::is_same<E, cx<R>>::value, "streamed rows carry values only");
  constexpr int NPOS = NQ + 2 * MD;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int R0 = G.R0;
  E* lf0 = reinterpret_cast<E*>(smem_raw);                                  // (RC + 2) rows
  E* lpk = ST ? reinterpret_cast<E*>(slots + (size_t)blockIdx.x * slot_len)  // MD x (RC + 1) rows
              : lf0 + (size_t)(G.RC + 2) * R0;
  E* sA = ST ? lf0 : lpk + (size_t)MD * (G.RC + 1) * R0;                   // A (NPOS x NPOS) then b (NPOS)
  const E* sb = sA + NPOS * NPOS;
  R* sq = reinterpret_cast<R*>(sA + NPOS * NPOS + NPOS);
  R* isq = sq + (kMaxCut + 4);
  for (int v = threadIdx.x; v < kMaxCut + 4; v += blockDim.x) {
    sq[v] = sqrt(R(v));
    isq[v] = v ? R(1) / sqrt(R(v)) : R(0);
  }
  for (int i = threadIdx.x; i < NPOS * NPOS + NPOS; i += blockDim.x) sA[i] = ET<E>::load(Ai + i, dT);
  // the unit's first unit_sync orders these LDS writes before their reads
  for (int w = blockIdx.x; w < nwork * G.nchunks; w += gridDim.x) {
    const int r = w / G.nchunks, c = w - r * G.nchunks;
    fwd_block_unit<MD, NQ, R, LevelPtrs<R>, E, ST, WV>(P, L, sA, sb, sq, isq, S, r, c, G, lf0, lpk, dT);
    if constexpr (WV > 1) __syncthreads();   // the next unit overwrites the rows
  }
}

template <int MD, int NQ, typename R, typename E, bool ST, int WV>
static void launch_fwd_block_w(size_t shm, int grid, hipStream_t st, const DevPlan& P, const LevelPtrs<R>& L,
                               const cx<R>* A, const cx<R>* b, int S, int nwork, const ChunkGeo& G, int64_t dT,
                               cx<R>* slots, int64_t slot_len) {
  if (shm > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_fwd_block<MD, NQ, R, E, ST, WV>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  hipLaunchKernelGGL((k_fwd_block<MD, NQ, R, E, ST, WV>), dim3(grid), dim3(kBT * WV), shm, st, P, L, A, b, S, nwork,
                     G, dT, slots, slot_len);
}
template <int MD, int NQ, typename R, typename E = cx<R>, bool ST = false>
static void launch_fwd_block_k(size_t shm, int grid, hipStream_t st, const DevPlan& P, const LevelPtrs<R>& L,
                               const cx<R>* A, const cx<R>* b, int S, int nwork, const ChunkGeo& G,
                               int64_t dT = 0, cx<R>* slots = nullptr, int64_t slot_len = 0) {
  // values with rows in LDS: kFwdWaves wavefronts per unit; the streamed
  // rows and the forward mode: one
  if constexpr (std::is_same<E, cx<R>>::value && !ST)
    launch_fwd_block_w<MD, NQ, R, E, ST, kFwdWaves>(shm, grid, st, P, L, A, b, S, nwork, G, dT, slots, slot_len);
  else
    launch_fwd_block_w<MD, NQ, R, E, ST, 1>(shm, grid, st, P, L, A, b, S, nwork, G, dT, slots, slot_len);
}

// Detected modes LO..LO + 3: values.
template <typename R, int LO>
hipError_t launch_fwd_block_range(const Plan& Pl, const DevPlan& P, int S, const LevelPtrs<R>& L, const cx<R>* A,
                                  const cx<R>* b, int nwork, hipStream_t st) {
  // a level with few units is latency-bound: halve the chunks to put more
  // wavefronts in flight; a large level keeps the full height
  const bool stm = Pl.st_fwd;
  ChunkGeo G = stm ? chunk_geo(Pl) : fwd_geo(Pl, nwork);
  if (stm && (int64_t)nwork * G.nchunks < kSmallLevelUnits) G = chunk_geo(Pl, kBT / 2);
  const size_t shm = stm ? fwd_stream_lds_bytes(Pl) : fwd_lds_bytes_for(Pl, G);
  if (shm > kMaxLds) return hipErrorInvalidConfiguration;
  // streamed rows: at most kStreamSlots workgroups, each with its slot after
  // the prep block
  const int grid = stm ? (int)std::min<int64_t>((int64_t)nwork * G.nchunks, kStreamSlots) : nwork * G.nchunks;
  cx<R>* slots = stm ? reinterpret_cast<cx<R>*>(reinterpret_cast<char*>(const_cast<cx<R>*>(A)) + prep_core_bytes(Pl))
                     : nullptr;
  const int64_t slen = (int64_t)fwd_stream_entries(Pl);
#define FD_LAUNCH_BLOCK_NQ(MDV, NQV)                                                                     \
  if (stm)                                                                                               \
    launch_fwd_block_k<MDV, NQV, R, cx<R>, true>(shm, grid, st, P, L, A, b, S, nwork, G, 0, slots, slen); \
  else                                                                                                   \
    launch_fwd_block_k<MDV, NQV, R>(shm, grid, st, P, L, A, b, S, nwork, G);
#define FD_LAUNCH_BLOCK(MDV)        \
  case MDV:                         \
    if (Pl.nq == 2) {               \
      FD_LAUNCH_BLOCK_NQ(MDV, 2)    \
    } else if (Pl.nq == 4) {        \
      FD_LAUNCH_BLOCK_NQ(MDV, 4)    \
    } else {                        \
      FD_LAUNCH_BLOCK_NQ(MDV, 6)    \
    }                               \
    break;
  switch (Pl.MD) {
    FD_LAUNCH_BLOCK(LO + 0)
    FD_LAUNCH_BLOCK(LO + 1)
    FD_LAUNCH_BLOCK(LO + 2)
    FD_LAUNCH_BLOCK(LO + 3)
    default:
      return hipErrorInvalidValue;
  }
#undef FD_LAUNCH_BLOCK
#undef FD_LAUNCH_BLOCK_NQ
  return hipGetLastError();
}

// ... values and tangents.
template <typename R, int LO>
hipError_t launch_jvp_block_range(const Plan& Pl, const DevPlan& P, int S, const LevelPtrs<R>& L, const cx<R>* A,
                                  const cx<R>* b, int nwork, int64_t dT, hipStream_t st) {
  ChunkGeo G = chunk_geo(Pl);
  if ((int64_t)nwork * G.nchunks < kSmallLevelUnits) G = chunk_geo(Pl, kBT / 2);
  const size_t shm = fwd_lds_bytes_for(Pl, G, true);
  if (shm > kMaxLds) return hipErrorInvalidConfiguration;   // rejected before the sweep
  const int grid = nwork * G.nchunks;
#define FD_LAUNCH_BLOCK_JVP(MDV)                                                                          \
  case MDV:                                                                                              \
    if (Pl.nq == 2)                                                                                      \
      launch_fwd_block_k<MDV, 2, R, dual<R>>(shm, grid, st, P, L, A, b, S, nwork, G, dT);            \
    else if (Pl.nq == 4)                                                                                 \
      launch_fwd_block_k<MDV, 4, R, dual<R>>(shm, grid, st, P, L, A, b, S, nwork, G, dT);            \
    else                                                                                                 \
      launch_fwd_block_k<MDV, 6, R, dual<R>>(shm, grid, st, P, L, A, b, S, nwork, G, dT);            \
    break;
  switch (Pl.MD) {
    FD_LAUNCH_BLOCK_JVP(LO + 0)
    FD_LAUNCH_BLOCK_JVP(LO + 1)
    FD_LAUNCH_BLOCK_JVP(LO + 2)
    FD_LAUNCH_BLOCK_JVP(LO + 3)
    default:
      return hipErrorInvalidValue;
  }
#undef FD_LAUNCH_BLOCK_JVP
  return hipGetLastError();
}

}  // namespace fd
