// Batched forward sweep: many independent circuits of uneven shape (mode
// count, cutoffs, detected/undetected split), level by level together.
//
// All pivots of one weight are independent (Sec. 2.2) and circuits are
// independent of each other, so step S of every circuit of one class (Algorithm
// 1 or 2, detected-mode count, block coordinates, parity) is one launch whose
// workgroups take (circuit, unit range) items from a table built with the
// schedule; the classes run on a few streams side by side.  Units are the
// device functions of the per-circuit level kernels, so the outputs are
// theirs bit for bit.
//
// The kernel boundary orders one step's writes before the next step's reads.
// A persistent cooperative grid with a device-wide barrier per step was
// measured and dropped: it inlines every unit shape, so it ran at two
// wavefronts per SIMD with one-wavefront units, and 48 circuits of 3 to 5 modes
// (9.3 GB of reads and writes) took 8.4 ms in it.
#pragma once

#include "fwd_units.h"

namespace fd {

constexpr int kOutIter = 8;                 // output elements per thread of the batched permutation

template <typename R>
struct BatchCirc {
  DevPlan P;
  PrepArgs pa;
  int wmax;                    // highest weight of the undetected block fill
  cx<R>* fam[kMaxFam];         // ring base of every family (index 0 unused)
  int64_t fstride[kMaxFam];    // ring slot stride in elements
  cx<R>* f0;                   // F0 at every level (the outputs in node order)
  cx<R>* Ai;                   // interleaved symmetrised A (npos x npos), then b, then c
  const cx<R>* A;
  const cx<R>* b;
  const cx<R>* c;
  cx<R>* rho;
  const uint64_t* mtab;        // digits of the lattice points (Algorithm 1), may be null
  const int* elist;
  const int* woff;
  int* status;
  int64_t out_elems, N;        // output elements; nodes (prod of detected cutoffs)
};

// Pointers the level kernels load from memory are generic to the compiler, which
// then emits flat loads and stores (counted by both the vector-memory and the
// LDS wait counters, so LDS waits also wait for HBM traffic).  They all point
// into device global memory: say so, and the accesses become global ones.
template <typename T>
using gptr = __attribute__((address_space(1))) T*;
// Loads a pointer stored at `slot` as a global-address-space pointer.
template <typename T>
__device__ __forceinline__ T* load_global(T* const* slot) {
  return (T*)(*reinterpret_cast<const gptr<T>*>(slot));
}

// Family pointers of one circuit at one level, computed from the ring bases.
template <typename R>
struct BatchRing {
  const BatchCirc<R>* __restrict__ C;
  int par;
  __device__ __forceinline__ cx<R>* operator[](int f) const {
    return load_global(&C->fam[f]) + (par ? C->fstride[f] : 0);
  }
};
template <typename R>
struct BatchLevel {
  BatchRing<R> rd, wr;
  const cx<R>* f0cur;
  cx<R>* f0nxt;
  const int* node;
};

template <typename R>
__device__ __forceinline__ BatchLevel<R> batch_level(const BatchCirc<R>* __restrict__ C, int S) {
  BatchLevel<R> L;
  L.rd.C = C;
  L.rd.par = (S - 1) & 1;
  L.wr.C = C;
  L.wr.par = S & 1;
  const int64_t* lvl = load_global(&C->P.lvl);
  const size_t B = (size_t)C->P.B;
  cx<R>* f0 = load_global(&C->f0);
  L.f0cur = f0 + (size_t)lvl[S] * B;
  L.f0nxt = S < C->P.smax ? f0 + (size_t)lvl[S + 1] * B : nullptr;
  const int* node = load_global(&C->P.node);
  L.node = node ? node + (size_t)lvl[S] * kNodeStride : nullptr;
  return L;
}

// One launch: step S of the circuits of one class (kind 0: Algorithm 1, 1:
// Algorithm 2), `nitems` workgroups.
struct BatchLaunch {
  int kind, MD, nq, odd;
  const void* circs;
  const BatchItem* items;
  int nitems, S;
  size_t shm;
};
// kernels_batch_level.hip
template <typename R>
hipError_t launch_batch_level(const BatchLaunch& a, hipStream_t st);

}  // namespace fd
