// Driver of the forward sweep (gfx950): one launch per step S (all targets of
// one step are independent, Sec. 2.2) around the prep, the undetected-block fill
// and the output permutation, which are here.  The level kernels are in
// kernels_point.hip (pt_units.h) and fwd_block.h (fwd_units.h).
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "fwd_units.h"

namespace fd {

template <typename R>
__global__ void k_prep(const cx<R>* __restrict__ A, const cx<R>* __restrict__ b, const cx<R>* __restrict__ c,
                       cx<R>* __restrict__ Ai, cx<R>* __restrict__ bi, cx<R>* __restrict__ ci,
                       cx<R>* __restrict__ f0node0, PrepArgs a, int* status) {
  prep_body<R>(A, b, c, Ai, bi, ci, f0node0, a, status);
}

// Step 1 of Algorithm 2: one wavefront, the undetected block in LDS (with
// E = dual<R>: values and tangents, the tangents dT bytes after the values).
template <typename R, int NQ, typename E = cx<R>, bool ST = false>
__global__ __launch_bounds__(64) void k_ufill(DevPlan P, const cx<R>* __restrict__ Ai,
                                              const cx<R>* __restrict__ bi, cx<R>* G,
                                              const int* __restrict__ elist, const int* __restrict__ woff,
                                              int wmax, int64_t dT) {
  if constexpr (NQ == 2) {
    ufill_rows_body<R, E>(P, Ai, bi, G, dT);
  } else {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    ufill_body<R, NQ, E, ST>(P, Ai, bi, G, elist, woff, wmax, reinterpret_cast<E*>(smem_raw), dT);
  }
}

// F0 (level-major nodes of B entries) -> rho, C order [kappa][n_D].
template <typename R, int EPT>
__global__ __launch_bounds__(kThreads) void k_out_perm(DevPlan P, const cx<R>* __restrict__ f0,
                                                       cx<R>* __restrict__ rho, int64_t N, int64_t total,
                                                       int* status) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  int* spn = reinterpret_cast<int*>(smem_raw);
  int64_t* slv = reinterpret_cast<int64_t*>(smem_raw + 16 * ((((P.MD + 1) * P.pnw) * 4 + 15) / 16));
  const int npn = (P.MD + 1) * P.pnw;
  for (int i = threadIdx.x; i < npn; i += blockDim.x) spn[i] = P.pn[i];
  for (int i = threadIdx.x; i <= P.smax; i += blockDim.x) slv[i] = P.MD > 0 ? P.lvl[i] : 0;
  __syncthreads();
  int bad = 0;
  if (P.B > 1) {
    cx<R>* tl = reinterpret_cast<cx<R>*>(reinterpret_cast<unsigned char*>(slv) + 16 * (((P.smax + 2) * 8 + 15) / 16));
    const int64_t tiles = ((N + kOutTN - 1) / kOutTN) * ((P.B + kOutTK - 1) / kOutTK);
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) bad |= out_perm_tile<R>(P, spn, slv, f0, rho, N, t, tl);
  } else {
    for (int64_t i0 = (int64_t)blockIdx.x * kThreads * EPT; i0 < total;
         i0 += (int64_t)gridDim.x * kThreads * EPT) {
      cx<R> v[EPT];
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        v[e] = out_perm_elem<R>(P, spn, slv, f0, N, min(i0 + e * kThreads + threadIdx.x, total - 1));
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int64_t idx = i0 + e * kThreads + threadIdx.x;
        if (idx >= total) break;
        if (!isfinite(v[e].x) || !isfinite(v[e].y)) bad = 1;
        st(rho + idx, v[e]);
      }
    }
  }
  if (bad) atomicOr(status, 1);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
// Block levels, compiled in eight translation units (precision, detected modes
// LO..LO + 3; values, values and tangents).
template <typename R, int LO>
hipError_t launch_fwd_block_range(const Plan& Pl, const DevPlan& P, int S, const LevelPtrs<R>& L, const cx<R>* A,
                                  const cx<R>* b, int nwork, hipStream_t st);
template <typename R, int LO>
hipError_t launch_jvp_block_range(const Plan& Pl, const DevPlan& P, int S, const LevelPtrs<R>& L, const cx<R>* A,
                                  const cx<R>* b, int nwork, int64_t dT, hipStream_t st);

// The undetected-block fill for the plan's number of block coordinates.
template <typename R>
static hipError_t launch_ufill(const Plan& Pl, const DevPlan& P, const cx<R>* Ai, const cx<R>* bi, cx<R>* f0,
                               hipStream_t st) {
  const size_t shm = ufill_launch_lds_bytes(Pl, false);
  if (shm > kMaxLds) return hipErrorInvalidConfiguration;
  auto* kfn = Pl.nq == 2 ? &k_ufill<R, 2>
              : Pl.st_ufill ? (Pl.nq == 4 ? &k_ufill<R, 4, cx<R>, true> : &k_ufill<R, 6, cx<R>, true>)
                            : (Pl.nq == 4 ? &k_ufill<R, 4> : &k_ufill<R, 6>);
  if (shm > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)shm);
  hipLaunchKernelGGL(kfn, dim3(1), dim3(64), shm, st, P, Ai, bi, f0, Pl.d_elist, Pl.d_woff, Pl.wmax, (int64_t)0);
  return hipGetLastError();
}

template <typename R>
static hipError_t launch_fwd_level_t(const Plan& Pl, const DevPlan& P, bool odd, int S, const LevelPtrs<R>& L,
                                     const void* Ai, const void* bi, hipStream_t st) {
  const int MD = Pl.MD;
  if (MD == 0) return hipSuccess;
  const int nwork = (int)Pl.ncnt[S];   // lattice points of level S
  if (nwork <= 0) return hipSuccess;
  const cx<R>* A = reinterpret_cast<const cx<R>*>(Ai);
  const cx<R>* b = reinterpret_cast<const cx<R>*>(bi);
  if (Pl.B == 1) {
    return launch_fwd_point_level<R>(Pl, P, odd, S, L, A, b, st);
  }
  return MD <= 4 ? launch_fwd_block_range<R, 1>(Pl, P, S, L, A, b, nwork, st)
                 : launch_fwd_block_range<R, 5>(Pl, P, S, L, A, b, nwork, st);
}

// Node-0 pointer of family f of group g at level S.
template <typename R>
static cx<R>* fam_level_ptr(const Plan& Pl, char* base, size_t off, int g, int S, bool ring) {
  if (S < 0) return nullptr;
  const size_t eb = sizeof(cx<R>);
  size_t node = ring ? (size_t)(S & 1) * Pl.maxN[g] : (size_t)Pl.lvl[(size_t)g * (Pl.smax + 2) + S];
  return reinterpret_cast<cx<R>*>(base + off + node * Pl.B * eb);
}

hipError_t launch_fwd_level(const Plan& Pl, bool odd, int S, const void* const* rd, void* const* wr,
                            const void* f0cur, void* f0nxt, const void* Ai, const void* bi, hipStream_t st) {
  if (!f0cur || !Ai || !bi) return hipErrorInvalidValue;   // read by every unit
  const DevPlan P = make_devplan(Pl, odd);
  if (Pl.dt == FD_C64) {
    LevelPtrs<float> L;
    std::memset(&L, 0, sizeof(L));
    for (int f = 1; f < Pl.nfam; ++f) {
      L.rd[f] = static_cast<const cx<float>*>(rd[f]);
      L.wr[f] = static_cast<cx<float>*>(wr[f]);
    }
    L.f0cur = static_cast<const cx<float>*>(f0cur);
    L.f0nxt = static_cast<cx<float>*>(f0nxt);
    L.node = Pl.d_node ? Pl.d_node + (size_t)Pl.lvl[S] * kNodeStride : nullptr;
    return launch_fwd_level_t<float>(Pl, P, odd, S, L, Ai, bi, st);
  }
  LevelPtrs<double> L;
  std::memset(&L, 0, sizeof(L));
  for (int f = 1; f < Pl.nfam; ++f) {
    L.rd[f] = static_cast<const cx<double>*>(rd[f]);
    L.wr[f] = static_cast<cx<double>*>(wr[f]);
  }
  L.f0cur = static_cast<const cx<double>*>(f0cur);
  L.f0nxt = static_cast<cx<double>*>(f0nxt);
  L.node = Pl.d_node ? Pl.d_node + (size_t)Pl.lvl[S] * kNodeStride : nullptr;
  return launch_fwd_level_t<double>(Pl, P, odd, S, L, Ai, bi, st);
}

// Copy of one level of every family (a checkpoint before its segment, for the
// one-workgroup reverse sweep, which takes a segment in one piece):
// family blockIdx.y, n[f] 16-byte (complex128) or 8-byte entries.
struct CopyFams {
  const void* src[kMaxFam];
  void* dst[kMaxFam];
  int64_t n[kMaxFam];
};

template <typename R>
__global__ __launch_bounds__(kThreads) void k_copy_fams(CopyFams a) {
  const int f = blockIdx.y;
  const cx<R>* src = static_cast<const cx<R>*>(a.src[f]);
  cx<R>* dst = static_cast<cx<R>*>(a.dst[f]);
  if (!src) return;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n[f]; i += (int64_t)gridDim.x * blockDim.x)
    st(dst + i, ld(src + i));
}

hipError_t launch_copy_fams(const Plan& Pl, const void* const* src, void* const* dst, const int64_t* n,
                            hipStream_t st) {
  CopyFams a;
  std::memset(&a, 0, sizeof(a));
  int64_t nmax = 0;
  for (int f = 0; f < Pl.nfam; ++f) {
    a.src[f] = src[f];
    a.dst[f] = dst[f];
    a.n[f] = src[f] ? n[f] : 0;
    nmax = std::max(nmax, a.n[f]);
  }
  if (nmax == 0) return hipSuccess;
  const unsigned gx = (unsigned)std::min<int64_t>((nmax + kThreads - 1) / kThreads, 1024);
  if (Pl.dt == FD_C64)
    hipLaunchKernelGGL((k_copy_fams<float>), dim3(gx, Pl.nfam), dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL((k_copy_fams<double>), dim3(gx, Pl.nfam), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_prep(const Plan& Pl, const void* A, const void* b, const void* c, void* Ai, void* f0node0,
                       hipStream_t st) {
  PrepArgs pa;
  std::memset(&pa, 0, sizeof(pa));
  for (int p = 0; p < Pl.npos; ++p) pa.pos2blk[p] = Pl.pos2blk[p];
  pa.npos = Pl.npos;
  pa.M2 = 2 * Pl.M;
  pa.check_b_zero = (Pl.flags == FD_B_ZERO) ? 1 : 0;
  const size_t n2 = (size_t)Pl.npos * Pl.npos;
  if (Pl.dt == FD_C64) {
    cx<float>* a = reinterpret_cast<cx<float>*>(Ai);
    hipLaunchKernelGGL((k_prep<float>), dim3(1), dim3(kThreads), 0, st, reinterpret_cast<const cx<float>*>(A),
                       reinterpret_cast<const cx<float>*>(b), reinterpret_cast<const cx<float>*>(c), a, a + n2,
                       a + n2 + Pl.npos, reinterpret_cast<cx<float>*>(f0node0), pa, Pl.d_status);
  } else {
    cx<double>* a = reinterpret_cast<cx<double>*>(Ai);
    hipLaunchKernelGGL((k_prep<double>), dim3(1), dim3(kThreads), 0, st, reinterpret_cast<const cx<double>*>(A),
                       reinterpret_cast<const cx<double>*>(b), reinterpret_cast<const cx<double>*>(c), a, a + n2,
                       a + n2 + Pl.npos, reinterpret_cast<cx<double>*>(f0node0), pa, Pl.d_status);
  }
  return hipGetLastError();
}

// Plans with a total photon cutoff return F0 in level order: a copy with the
// non-finite check.
template <typename R>
__global__ __launch_bounds__(kThreads) void k_copy_levels(const cx<R>* __restrict__ f0, cx<R>* __restrict__ rho,
                                                          int64_t n, int* status) {
  int bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const cx<R> v = ld(f0 + i);
    if (!isfinite(v.x) || !isfinite(v.y)) bad = 1;
    st(rho + i, v);
  }
  if (bad) atomicOr(status, 1);
}

// Partial masses of level S = S0 + blockIdx.y (the sum of Re F0, i.e. of the
// detection probabilities of the level): part blockIdx.x of kMassParts
// contiguous chunks, strided per-thread sums, then a fixed-order tree;
// mass[S * kMassParts + part].
template <typename R>
__global__ __launch_bounds__(kThreads) void k_level_mass(const cx<R>* __restrict__ f0, const int64_t* __restrict__ lvl,
                                                         int S0, double* mass) {
  __shared__ double red[kThreads];
  const int S = S0 + blockIdx.y;
  const int64_t n = lvl[S + 1] - lvl[S];
  const int64_t chunk = (n + kMassParts - 1) / kMassParts;
  const int64_t i0 = lvl[S] + (int64_t)blockIdx.x * chunk;
  const int64_t i1 = min(lvl[S + 1], i0 + chunk);
  double acc = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) acc += (double)ld(f0 + i).x;
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) mass[(size_t)S * kMassParts + blockIdx.x] = red[0];
}

template <typename R>
__global__ __launch_bounds__(kThreads) void k_clear(cx<R>* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    st(p + i, czero<R>());
}

// F0 in node order -> rho (C order), with the non-finite check.
template <typename R>
static hipError_t launch_out_perm_t(const Plan& Pl, const DevPlan& P, const cx<R>* f0, void* rho, hipStream_t st) {
  if (Pl.level_cap >= 0) {
    const int64_t n = Pl.nodes_total;
    KTimer kt(Pl, KK_OUT_PERM, st);
    hipLaunchKernelGGL((k_copy_levels<R>), dim3((unsigned)std::min<int64_t>((n + kThreads - 1) / kThreads, 65536)),
                       dim3(kThreads), 0, st, f0, reinterpret_cast<cx<R>*>(rho), n, Pl.d_status);
    return hipGetLastError();
  }
  const int64_t total = Pl.out_elems;
  const int64_t tiles = ((Pl.nodes_total + kOutTN - 1) / kOutTN) * ((Pl.B + kOutTK - 1) / kOutTK);
  const int ept = total >= kOutEPTMin ? kOutEPT : 1;
  const int64_t grid = std::min<int64_t>(Pl.B > 1 ? tiles : (total + kThreads * ept - 1) / (kThreads * ept), 65536);
  const size_t shm = 16 * ((((size_t)(Pl.MD + 1) * (Pl.smax + 3)) * 4 + 15) / 16) +
                     16 * (((size_t)(Pl.smax + 2) * 8 + 15) / 16) + (size_t)kOutTN * (kOutTK + 1) * sizeof(cx<R>);
  KTimer kt(Pl, KK_OUT_PERM, st);
  auto* kfn = ept == 1 ? &k_out_perm<R, 1> : &k_out_perm<R, kOutEPT>;
  hipLaunchKernelGGL(kfn, dim3(grid), dim3(kThreads), shm, st, P, f0, reinterpret_cast<cx<R>*>(rho),
                     (int64_t)Pl.nodes_total, total, Pl.d_status);
  return hipGetLastError();
}

// Forward sweep for a checkpointed reverse sweep: F0 at every level goes to
// the saved buffer, the other families run in a two-level ring (the first
// two slots of the segment buffer) except at the level just below each segment,
// which is written to its checkpoint and read there by the next level (copying
// these levels out of the ring and, in the reverse sweep, into the segment
// buffer took 1.09 of the 17.1 ms of five detected modes of cutoff 8 and an undetected one of
// cutoff 30 in segments of six levels).
template <typename R>
static hipError_t run_forward_ckpt_t(const Plan& Pl, bool odd, const void* A, const void* b, const void* c,
                                     void* rho, char* ws, char* saved, hipStream_t st) {
  const CkptLayout Lc = ckpt_layout(Pl);
  const SegLayout Sg = seg_layout(Pl);
  const size_t eb = sizeof(cx<R>);
  cx<R>* Ai = reinterpret_cast<cx<R>*>(ws);   // prep block at the start of the workspace
  cx<R>* bi = Ai + (size_t)Pl.npos * Pl.npos;
  cx<R>* f0 = reinterpret_cast<cx<R>*>(saved + Lc.f0);
  const DevPlan P = make_devplan(Pl, odd);
  hipError_t e;
  {
    KTimer kt(Pl, KK_PREP, st);
    e = launch_prep(Pl, A, b, c, Ai, f0, st);
  }
  if (e != hipSuccess) return e;
  if (Pl.B > 1) {
    KTimer kt(Pl, KK_UFILL, st);
    if ((e = launch_ufill<R>(Pl, P, Ai, bi, f0, st)) != hipSuccess) return e;
  }
  const int s = Pl.ckpt, MD = Pl.MD;
  auto used = [&](int f) { return ckpt_keeps_family(Pl, f) && (odd || f >= 1 + 2 * MD); };
  auto level = [&](int f, int S) -> char* {   // family f at level S
    if ((S + 1) % s == 0 && S < Pl.smax) return saved + Lc.ck[(size_t)((S + 1) / s - 1) * Pl.nfam + f];
    return ws + Sg.fam[f] + (size_t)(S & 1) * Pl.maxN[Pl.fam_group[f]] * Pl.B * eb;
  };
  for (int S = 0; S <= Pl.smax && MD > 0; ++S) {
    const void* rd[kMaxFam] = {};
    void* wr[kMaxFam] = {};
    for (int f = 1; f < Pl.nfam; ++f) {
      if (!used(f)) continue;
      rd[f] = S > 0 ? level(f, S - 1) : nullptr;
      wr[f] = level(f, S);
    }
    const cx<R>* f0cur = f0 + (size_t)Pl.lvl[S] * Pl.B;
    cx<R>* f0nxt = S < Pl.smax ? f0 + (size_t)Pl.lvl[S + 1] * Pl.B : nullptr;
    {
      KTimer kt(Pl, KK_FWD_LEVEL, st);
      e = launch_fwd_level(Pl, odd, S, rd, wr, f0cur, f0nxt, Ai, bi, st);
    }
    if (e != hipSuccess) return e;
  }
  if (!rho) return hipSuccess;
  return launch_out_perm_t<R>(Pl, P, f0, rho, st);
}

template <typename R>
static hipError_t run_forward_t(const Plan& Pl, bool odd, const void* A, const void* b, const void* c, void* rho,
                                char* ws, char* saved, hipStream_t st, StopRule* stop) {
  if (saved && Pl.ckpt > 0) return run_forward_ckpt_t<R>(Pl, odd, A, b, c, rho, ws, saved, st);
  const bool store_all = saved != nullptr;
  // prep lives in the workspace; intermediates in `saved` (store-all) or the workspace (ring)
  FwdLayout Lw = fwd_layout(Pl, odd, false, 0);
  FwdLayout Ls = fwd_layout(Pl, true, true, 0);
  char* fb = store_all ? saved : ws;
  const FwdLayout& LF = store_all ? Ls : Lw;
  cx<R>* Ai = reinterpret_cast<cx<R>*>(ws + Lw.prep);
  cx<R>* bi = Ai + (size_t)Pl.npos * Pl.npos;
  cx<R>* ci = bi + Pl.npos;
  cx<R>* f0 = reinterpret_cast<cx<R>*>(fb + LF.f0);
  DevPlan P = make_devplan(Pl, odd);
  if (store_all && Pl.wcnt) {   // debug write counters over the saved buffer
    P.wcnt = Pl.wcnt;
    P.wbase = saved;
    P.wcnt_n = (int64_t)Pl.wcnt_n;
  }
  (void)ci;
  hipError_t e;
  if (stop) {
    stop->levels_done = Pl.smax + 1;
    stop->mass = 0.0;
  }
  if (Pl.small_fwd && !stop) {
    void* fam[kMaxFam] = {};
    fam[0] = f0;
    for (int f = 1; f < Pl.nfam; ++f) fam[f] = LF.fam[f] ? fb + LF.fam[f] : nullptr;
    KTimer kt(Pl, KK_FWD_LEVEL, st);
    return launch_point_small_fwd<R>(Pl, P, odd, static_cast<const cx<R>*>(A), static_cast<const cx<R>*>(b),
                                     static_cast<const cx<R>*>(c), Ai, fam, !store_all, static_cast<cx<R>*>(rho), st);
  }
  {
    KTimer kt(Pl, KK_PREP, st);
    e = launch_prep(Pl, A, b, c, Ai, f0, st);
  }
  if (e != hipSuccess) return e;
  if (Pl.B > 1) {
    KTimer kt(Pl, KK_UFILL, st);
    if ((e = launch_ufill<R>(Pl, P, Ai, bi, f0, st)) != hipSuccess) return e;
  }
  for (int S = 0; S <= Pl.smax && Pl.MD > 0; ++S) {
    LevelPtrs<R> L;
    std::memset(&L, 0, sizeof(L));
    for (int f = 1; f < Pl.nfam; ++f) {
      if (LF.fam[f] == 0) continue;
      const int g = Pl.fam_group[f];
      L.rd[f] = fam_level_ptr<R>(Pl, fb, LF.fam[f], g, S - 1, !store_all);
      L.wr[f] = fam_level_ptr<R>(Pl, fb, LF.fam[f], g, S, !store_all);
    }
    L.f0cur = fam_level_ptr<R>(Pl, fb, LF.f0, 0, S, false);
    L.node = Pl.d_node ? Pl.d_node + (size_t)Pl.lvl[S] * kNodeStride : nullptr;
    L.f0nxt = S < Pl.smax ? fam_level_ptr<R>(Pl, fb, LF.f0, 0, S + 1, false) : nullptr;
    {
      KTimer kt(Pl, KK_FWD_LEVEL, st);
      e = launch_fwd_level_t<R>(Pl, P, odd, S, L, Ai, bi, st);
    }
    if (e != hipSuccess) return e;
    if (stop && ((S + 1) % kStopBlock == 0 || S == Pl.smax)) {
      // levels S0..S are final (F0 of a level is written by the launch below it)
      const int S0 = S - S % kStopBlock;
      hipLaunchKernelGGL((k_level_mass<R>), dim3(kMassParts, S - S0 + 1), dim3(kThreads), 0, st, f0, Pl.d_lvl, S0,
                         Pl.d_mass);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      double hm[kStopBlock * kMassParts];
      if ((e = hipMemcpyAsync(hm, Pl.d_mass + (size_t)S0 * kMassParts, (size_t)(S - S0 + 1) * kMassParts * sizeof(double),
                              hipMemcpyDeviceToHost, st)) != hipSuccess ||
          (e = hipStreamSynchronize(st)) != hipSuccess)
        return e;
      int hit = -1;
      for (int k = 0; k <= S - S0 && hit < 0; ++k) {
        double m = 0.0;
        for (int q = 0; q < kMassParts; ++q) m += hm[k * kMassParts + q];
        stop->mass += m;
        if (stop->mass >= 1.0 - stop->eps) hit = S0 + k;
      }
      if (hit >= 0) {
        stop->levels_done = hit + 1;
        const int64_t from = Pl.lvl[hit + 1], to = Pl.lvl[Pl.smax + 1];   // F0 above level hit
        if (to > from) {
          hipLaunchKernelGGL((k_clear<R>), dim3((unsigned)std::min<int64_t>((to - from + kThreads - 1) / kThreads, 65536)),
                             dim3(kThreads), 0, st, f0 + from, to - from);
          if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        break;
      }
    }
  }
  if (!rho) return hipSuccess;   // recompute for the reverse sweep: no output needed
  return launch_out_perm_t<R>(Pl, P, f0, rho, st);
}

hipError_t launch_out_perm(const Plan& Pl, const void* f0, void* rho, hipStream_t st) {
  const DevPlan P = make_devplan(Pl, false);
  if (Pl.dt == FD_C64) return launch_out_perm_t<float>(Pl, P, static_cast<const cx<float>*>(f0), rho, st);
  return launch_out_perm_t<double>(Pl, P, static_cast<const cx<double>*>(f0), rho, st);
}

hipError_t run_forward(const Plan& Pl, bool odd, const void* A, const void* b, const void* c, void* rho, void* ws,
                       void* saved, hipStream_t st, StopRule* stop) {
  if (Pl.dt == FD_C64)
    return run_forward_t<float>(Pl, odd, A, b, c, rho, (char*)ws, (char*)saved, st, stop);
  return run_forward_t<double>(Pl, odd, A, b, c, rho, (char*)ws, (char*)saved, st, stop);
}


// ---------------------------------------------------------------------------
// Forward mode (the tangent recurrences of Sec. 2.5, summed along one direction
// (dA, db, dc)): differentiating Eq. recrel gives, for a pivot p and write
// direction i,
//   sqrt(p_i + 1) dG_{p+1_i} = db_i G_p + b_i dG_p
//                              + sum_l sqrt(p_l) (dA_il G_{p-1_l} + A_il dG_{p-1_l}),
// with dG_0 = dc.  The tangents need exactly the reads and writes of the
// values, so every kept amplitude gets its tangent in a second workspace of
// the same layout, dT bytes further on, and the same lane carries both.
// ---------------------------------------------------------------------------
template <typename R>
static hipError_t run_jvp_t(const Plan& Pl, const void* A, const void* b, const void* c, const void* dA,
                            const void* db, const void* dc, void* rho, void* drho, char* ws, int64_t half,
                            hipStream_t st) {
  const FwdLayout Lw = fwd_layout(Pl, true, false, 0);
  char* wt = ws + half;
  cx<R>* Ai = reinterpret_cast<cx<R>*>(ws + Lw.prep);
  cx<R>* bi = Ai + (size_t)Pl.npos * Pl.npos;
  cx<R>* dAi = reinterpret_cast<cx<R>*>(wt + Lw.prep);
  cx<R>* dbi = dAi + (size_t)Pl.npos * Pl.npos;
  cx<R>* f0 = reinterpret_cast<cx<R>*>(ws + Lw.f0);
  cx<R>* tf0 = reinterpret_cast<cx<R>*>(wt + Lw.f0);
  const DevPlan P = make_devplan(Pl, true);
  hipError_t e;
  {
    KTimer kt(Pl, KK_PREP, st);
    if ((e = launch_prep(Pl, A, b, c, Ai, f0, st)) != hipSuccess) return e;
    if ((e = launch_prep(Pl, dA, db, dc, dAi, tf0, st)) != hipSuccess) return e;
  }
  if (Pl.B > 1) {
    // step 1 of Algorithm 2 with tangents
    KTimer kt(Pl, KK_UFILL, st);
    const size_t shm = ufill_jvp_lds_bytes(Pl);
    if (shm > kMaxLds) return hipErrorInvalidConfiguration;   // rejected before the sweep
    auto* kfn = Pl.nq == 2 ? &k_ufill<R, 2, dual<R>> : Pl.nq == 4 ? &k_ufill<R, 4, dual<R>> : &k_ufill<R, 6, dual<R>>;
    if (shm > 65536)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)shm);
    hipLaunchKernelGGL(kfn, dim3(1), dim3(64), shm, st, P, Ai, bi, f0, Pl.d_elist, Pl.d_woff, Pl.wmax, half);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  for (int S = 0; S <= Pl.smax && Pl.MD > 0; ++S) {
    const int nwork = (int)Pl.ncnt[S];
    if (nwork <= 0) continue;
    LevelPtrs<R> L;
    std::memset(&L, 0, sizeof(L));
    for (int f = 1; f < Pl.nfam; ++f) {
      if (Lw.fam[f] == 0) continue;
      const int g = Pl.fam_group[f];
      L.rd[f] = fam_level_ptr<R>(Pl, ws, Lw.fam[f], g, S - 1, true);
      L.wr[f] = fam_level_ptr<R>(Pl, ws, Lw.fam[f], g, S, true);
    }
    L.f0cur = fam_level_ptr<R>(Pl, ws, Lw.f0, 0, S, false);
    L.f0nxt = S < Pl.smax ? fam_level_ptr<R>(Pl, ws, Lw.f0, 0, S + 1, false) : nullptr;
    KTimer kt(Pl, KK_FWD_LEVEL, st);
    if (Pl.B > 1) {
      L.node = Pl.d_node + (size_t)Pl.lvl[S] * kNodeStride;
      e = Pl.MD <= 4 ? launch_jvp_block_range<R, 1>(Pl, P, S, L, Ai, bi, nwork, half, st)
                     : launch_jvp_block_range<R, 5>(Pl, P, S, L, Ai, bi, nwork, half, st);
      if (e != hipSuccess) return e;
      continue;
    }
    if ((e = launch_fwd_point_level<R>(Pl, P, true, S, L, Ai, bi, st, half)) != hipSuccess) return e;
  }
  if ((e = launch_out_perm_t<R>(Pl, P, f0, rho, st)) != hipSuccess) return e;
  return launch_out_perm_t<R>(Pl, P, tf0, drho, st);
}

hipError_t run_jvp(const Plan& Pl, const void* A, const void* b, const void* c, const void* dA, const void* db,
                   const void* dc, void* rho, void* drho, void* ws, hipStream_t st) {
  const int64_t half = (int64_t)jvp_half_bytes(Pl);
  if (Pl.dt == FD_C64) return run_jvp_t<float>(Pl, A, b, c, dA, db, dc, rho, drho, (char*)ws, half, st);
  return run_jvp_t<double>(Pl, A, b, c, dA, db, dc, rho, drho, (char*)ws, half, st);
}

}  // namespace fd
