// Whole sweeps of small plans with every mode detected in one workgroup: input
// prep, every level, the permutations and (reverse) the final sums in one launch.
//
// A level of a small lattice is a few 16-point tiles, so a launch per level costs
// its launch and its tables (3-6 us) for about 2 us of dependent loads and
// products, and a training step of 100 probabilities is some 45 launches.  One
// workgroup runs the levels with a barrier between them instead; its wavefronts
// share a CU, so its L1 and a workgroup barrier order one level's writes before
// the next level's reads.  The tiles are those of the level kernels (pt_units.h,
// vjp_point_units.h), so the amplitudes are theirs bit for bit.  Which plans:
// kSmallFwdItems, kSmallVjpItems in fd_internal.h.
#include <algorithm>
#include <cstring>

#include "vjp_point_units.h"

namespace fd {

// sixteen wavefronts forward (128 registers each), eight in the reverse (256)
constexpr int kSmallFwdThreads = 1024, kSmallFwdWaves = kSmallFwdThreads / 64;
constexpr int kSmallThreads = 512, kSmallWaves = kSmallThreads / 64;

// Family arrays of a sweep: node-0 pointers, and whether they are two-level
// rings or hold every level.
template <typename R>
struct SmallFams {
  cx<R>* f[kMaxFam];
  int ring;
};
// ... at one level; grp: group of each family (LDS).
template <typename R>
struct SmallLevel {
  const SmallFams<R>& F;
  const DevPlan& P;
  const unsigned char* grp;
  int S;
  __device__ __forceinline__ cx<R>* operator[](int f) const {
    if (S < 0) return F.f[f];   // no such level: never dereferenced
    const int g = grp[f];
    return F.f[f] + (F.ring ? (S & 1) * P.ringN[g] : P.lvl[g * (P.smax + 2) + S]);
  }
};

template <int MD>
__device__ __forceinline__ void small_groups(unsigned char* grp) {
  for (int f = threadIdx.x; f < 1 + 3 * MD + MD * (MD - 1); f += blockDim.x) {
    int g = 0;
    if (f >= 1 + 3 * MD) {
      int q = (f - 1 - 3 * MD) >> 1;   // pair index: (g, j) row by row
      while (q >= MD - 1 - g) q -= MD - 1 - g++;
    } else if (f >= 1 + 2 * MD) {
      g = f - 1 - 2 * MD;
    }
    grp[f] = (unsigned char)g;
  }
}

template <typename R>
struct SmallFwd {
  SmallFams<R> fam;   // fam.f[0] = F0 (every level)
  const cx<R>*A, *b, *c;
  cx<R>*Ai, *rho;     // rho null: no output wanted
  const uint64_t* mt;
  PrepArgs pa;
  int* status;
  int level_order;    // output in level order (a total photon cutoff)
};

// Which levels a sweep takes: the even ones (b = 0), all, or as b says -- read
// on the device, so that a call need not wait for its stream and read b first.
enum SmallMode { kSmallEven = 0, kSmallAll = 1, kSmallByB = 2 };
template <typename R>
__device__ __forceinline__ bool b_is_zero(const cx<R>* b, int n) {
  int nz = 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const cx<R> v = ld(b + i);
    nz |= !(v.x == R(0) && v.y == R(0));   // (a NaN is not zero)
  }
  return __syncthreads_or(nz) == 0;
}

template <int MD, bool ODD, typename R>
__device__ __forceinline__ void point_small_fwd(const DevPlan& P, const SmallFwd<R>& a, unsigned char* smem_raw) {
  constexpr int NT = pt_table_entries(MD);
  R* sq = reinterpret_cast<R*>(smem_raw);
  uint64_t* tab = reinterpret_cast<uint64_t*>(sq + 2 * (kMaxCut + 4));   // two levels x (read, write)
  int64_t* slv = reinterpret_cast<int64_t*>(tab + 4 * NT);
  int* rows = reinterpret_cast<int*>(slv + P.smax + 2);
  int* spn = rows + kSmallFwdWaves * pt_row_ints(MD, 1);
  unsigned char* grp = reinterpret_cast<unsigned char*>(spn + (MD + 1) * P.pnw);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  rows += wave * pt_row_ints(MD, 1);
  cx<R>* bi = a.Ai + 4 * MD * MD;
  cx<R>* f0 = a.fam.f[0];
  prep_body<R>(a.A, a.b, a.c, a.Ai, bi, bi + 2 * MD, f0, a.pa, a.status);
  pt_load_tables<R>(P, MD, sq, spn);
  small_groups<MD>(grp);
  for (int S = threadIdx.x; S < P.smax + 2; S += blockDim.x) slv[S] = P.lvl[S];
  __syncthreads();
  struct {
    SmallLevel<R> rd, wr;
    const cx<R>* f0cur;
    cx<R>* f0nxt;
  } L{{a.fam, P, grp, 0}, {a.fam, P, grp, 0}, nullptr, nullptr};
  auto fill = [&](int S) {
    L.rd.S = S - 1;
    L.wr.S = S;
    L.f0cur = f0 + slv[S];
    L.f0nxt = f0 + slv[S + 1];
    uint64_t* t = tab + (S & 1) * 2 * NT;
    pt_fill_pointers<MD, ODD, R>(L, t, t + NT);
  };
  PtConst<MD, ODD, false, R> C;
  C.load(P, a.Ai, bi, 0);
  fill(0);
  __syncthreads();
  for (int S = 0; S <= P.smax; ++S) {
    if (S < P.smax) fill(S + 1);   // the other table
    uint64_t* t = tab + (S & 1) * 2 * NT;
    const PtLds<R> Y{sq, sq + (kMaxCut + 4), spn, t, t + NT};
    PtItems I;
#pragma unroll
    for (int K = 0; K < MD; ++K) I.n[K] = (int)(P.lvl[K * (P.smax + 2) + S + 1] - P.lvl[K * (P.smax + 2) + S]);
    for (int u = wave;; u += kSmallFwdWaves) {
      int K = 0, base = 0, n = 0;
      if (!pt_item<MD>(I, u, &K, &base, &n)) break;
      fwd_point_item<MD, ODD, false, R>(P, Y, C, f0 + slv[S], S < P.smax, a.mt + slv[S], S, K, base, n, rows);
    }
    __syncthreads();
  }
  if (!a.rho) return;
  const int n = (int)slv[P.smax + 1];
  int bad = 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const cx<R> v = ld(f0 + (a.level_order ? i : node_of_cindex(P, spn, slv, i)));
    if (!isfinite(v.x) || !isfinite(v.y)) bad = 1;
    st(a.rho + i, v);
  }
  if (bad) atomicOr(a.status, 1);
}

template <int MD, int MODE, typename R>
__global__ __launch_bounds__(kSmallFwdThreads) void k_point_small_fwd(DevPlan P, SmallFwd<R> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (MODE == kSmallEven || (MODE == kSmallByB && b_is_zero(a.b, a.pa.M2)))
    point_small_fwd<MD, false, R>(P, a, smem_raw);
  else
    point_small_fwd<MD, true, R>(P, a, smem_raw);
}

template <typename R>
struct SmallVjp {
  SmallFams<R> fam;    // forward values, every level (f[0] = F0)
  SmallFams<R> gfam;   // cotangent rings (f[0] = F0)
  const cx<R>*A, *b, *c, *drho;
  cx<R>*Ai, *g0, *dA, *db, *dc;   // g0: drho in node order
  const uint64_t* mt;
  PrepArgs pa;
  int blk2pos[2 * kMaxModes];
  int* status;
  int level_order;     // a total photon cutoff: drho in level order, no level above the last
  // the levels of this launch, from the top (a checkpointed sweep: one segment
  // of levels per launch, the running sums kept in `state` between them)
  int hi, lo;
  double* state;
};

template <int MD, bool ODD, typename R>
__device__ __forceinline__ void point_small_vjp(const DevPlan& P, const SmallVjp<R>& a, unsigned char* smem_raw) {
  constexpr int NE = pt_vjp_entries(MD), NT = pt_table_entries(MD), NP = 2 * MD, NR = NP + 1, NPAIR = NP * NR;
  R* sq = reinterpret_cast<R*>(smem_raw);
  uint64_t* tab = reinterpret_cast<uint64_t*>(sq + 2 * (kMaxCut + 4));   // two levels
  cx<R>* turn = reinterpret_cast<cx<R>*>(tab + 2 * NE);
  int64_t* slv = reinterpret_cast<int64_t*>(turn + kSmallWaves * kPtPos * kTurn);
  int* rows = reinterpret_cast<int*>(slv + P.smax + 2);
  int* spn = rows + kSmallWaves * pt_row_ints(MD, 1);
  unsigned char* grp = reinterpret_cast<unsigned char*>(spn + (MD + 1) * P.pnw);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  turn += wave * kPtPos * kTurn;
  rows += wave * pt_row_ints(MD, 1);
  cx<R>* bi = a.Ai + 4 * MD * MD;
  const bool top = a.hi == P.smax;
  if (top) prep_body<R>(a.A, a.b, a.c, a.Ai, bi, bi + 2 * MD, (cx<R>*)nullptr, a.pa, a.status);
  pt_load_tables<R>(P, MD, sq, spn);
  small_groups<MD>(grp);
  for (int S = threadIdx.x; S < P.smax + 2; S += blockDim.x) slv[S] = P.lvl[S];
  __syncthreads();
  const int n = top ? (int)slv[P.smax + 1] : 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    st(a.g0 + (a.level_order ? i : node_of_cindex(P, spn, slv, i)), ld(a.drho + i));
  if (top && a.level_order)   // the families of the last level feed no target
    for (int f = ODD ? 1 : 1 + 2 * MD; f < 1 + 3 * MD + MD * (MD - 1); ++f) {
      cx<R>* p = SmallLevel<R>{a.gfam, P, grp, P.smax}[f];
      for (int i = threadIdx.x; i < (int)P.ringN[grp[f]]; i += blockDim.x) st(p + i, czero<R>());
    }
  struct {
    SmallLevel<R> fprev, fcur, gprev, gcur;
    const cx<R>* gf0nxt;
  } V{{a.fam, P, grp, 0}, {a.fam, P, grp, 0}, {a.gfam, P, grp, 0}, {a.gfam, P, grp, 0}, nullptr};
  auto fill = [&](int S) {
    V.fprev.S = V.gprev.S = S - 1;
    V.fcur.S = V.gcur.S = S;
    V.gf0nxt = a.gfam.f[0] + ((S + 1) & 1) * P.ringN[0];
    uint64_t* t = tab + (S & 1) * NE;
    pt_fill_vjp_pointers<MD, ODD, R>(V, t, t + NT, t + 2 * NT);
  };
  VjpPtConst<MD, ODD, R> C;
  C.load(P, a.Ai, bi);
  VjpPtSums<MD, R> Z;
  Z.zero();
  // (a thread's sums, at stride kSmallThreads)
  constexpr int NS = 12 + 2 * PtMat<MD, R>::KS;
  auto sum_at = [&](int i) -> double& { return a.state[(size_t)i * kSmallThreads + threadIdx.x]; };
  if (!top) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Z.acc.p1[0][j] = sum_at(j);
      Z.acc.p2[0][j] = sum_at(4 + j);
      Z.acc.p3[0][j] = sum_at(8 + j);
    }
#pragma unroll
    for (int s = 0; s < PtMat<MD, R>::KS; ++s) {
      Z.bx[s] = sum_at(12 + 2 * s);
      Z.by[s] = sum_at(13 + 2 * s);
    }
  }
  static_assert((size_t)NS * kSmallThreads * 8 <= (size_t)kPartialSlots * NP * NR * 16, "the sums fit the slots");
  fill(a.hi);
  __syncthreads();
  for (int S = a.hi; S >= a.lo; --S) {
    if (S > a.lo) fill(S - 1);   // the other table
    uint64_t* t = tab + (S & 1) * NE;
    const VjpPtLevel<R> L{t,
                          t + NT,
                          t + 2 * NT,
                          sq,
                          sq + (kMaxCut + 4),
                          spn,
                          a.fam.f[0] + slv[S],
                          a.g0 + slv[S],
                          a.gfam.f[0] + (S & 1) * P.ringN[0],
                          !(a.level_order && S == P.smax)};
    const int nw = (int)(slv[S + 1] - slv[S]);
    for (int base = 16 * wave; base < nw; base += 16 * kSmallWaves)
      vjp_point_tile<MD, ODD, 1, R>(P, L, C, Z, a.mt + slv[S], S, base, nw, turn, rows);
    __syncthreads();
  }
  if (a.lo > 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sum_at(j) = Z.acc.p1[0][j];
      sum_at(4 + j) = Z.acc.p2[0][j];
      sum_at(8 + j) = Z.acc.p3[0][j];
    }
#pragma unroll
    for (int s = 0; s < PtMat<MD, R>::KS; ++s) {
      sum_at(12 + 2 * s) = Z.bx[s];
      sum_at(13 + 2 * s) = Z.by[s];
    }
    return;
  }
  // the wavefronts' pair tables in order, then the caller's block order
  // (symmetric part of Abar, zero for dropped modes)
  cx<double>* red = reinterpret_cast<cx<double>*>(smem_raw);
  Z.template store<ODD>(red + (size_t)wave * NPAIR);
  __syncthreads();
  auto pair = [&](int i, int l) -> cx<double> {
    double x = 0.0, y = 0.0;
    for (int w = 0; w < kSmallWaves; ++w) {
      x += red[w * NPAIR + i * NR + l].x;
      y += red[w * NPAIR + i * NR + l].y;
    }
    return cmake<double>(x, y);
  };
  const int M2 = a.pa.M2;
  for (int i = threadIdx.x; i < M2 * M2; i += blockDim.x) {
    const int p = a.blk2pos[i / M2], q = a.blk2pos[i % M2];
    cx<double> v = czero<double>();
    if (p >= 0 && q >= 0) v = cscale(cadd(pair(p, q), pair(q, p)), 0.5);
    st(a.dA + i, cmake<R>((R)v.x, (R)v.y));
  }
  for (int i = threadIdx.x; i < M2; i += blockDim.x) {
    const int p = a.blk2pos[i];
    cx<double> v = czero<double>();
    if (ODD && p >= 0) v = pair(p, NP);
    st(a.db + i, cmake<R>((R)v.x, (R)v.y));
  }
  if (threadIdx.x == 0) st(a.dc, ld(a.gfam.f[0]));
}

template <int MD, int MODE, typename R>
__global__ __launch_bounds__(kSmallThreads) void k_point_small_vjp(DevPlan P, SmallVjp<R> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  if (MODE == kSmallEven || (MODE == kSmallByB && b_is_zero(a.b, a.pa.M2)))
    point_small_vjp<MD, false, R>(P, a, smem_raw);
  else
    point_small_vjp<MD, true, R>(P, a, smem_raw);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
static void small_prep(const Plan& Pl, PrepArgs* pa) {
  std::memset(pa, 0, sizeof(*pa));
  for (int p = 0; p < Pl.npos; ++p) pa->pos2blk[p] = Pl.pos2blk[p];
  pa->npos = Pl.npos;
  pa->M2 = 2 * Pl.M;
  pa->check_b_zero = Pl.flags == FD_B_ZERO ? 1 : 0;
}
// level offsets, rank rows, PN table, family groups
static size_t small_tail_lds(const Plan& Pl, int waves) {
  return (size_t)(Pl.smax + 2) * 8 + (size_t)waves * pt_row_ints(Pl.MD, 1) * 4 +
         (size_t)(Pl.MD + 1) * (Pl.smax + 3) * 4 + kMaxFam;
}

#define FD_SMALL(KERN, THREADS)                                                                                       \
  {                                                                                                                \
    if (shm > 65536)                                                                                               \
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&KERN), hipFuncAttributeMaxDynamicSharedMemorySize,  \
                                (int)shm);                                                                         \
    hipLaunchKernelGGL(KERN, dim3(1), dim3(THREADS), shm, st, P, a);                                               \
  }
#define FD_SMALL_CASE(NAME, THREADS, MDV)                     \
  case MDV:                                                   \
    if (by_b)                                                 \
      FD_SMALL((NAME<MDV, kSmallByB, R>), THREADS)            \
    else if (odd)                                             \
      FD_SMALL((NAME<MDV, kSmallAll, R>), THREADS)            \
    else                                                      \
      FD_SMALL((NAME<MDV, kSmallEven, R>), THREADS)           \
    break;
#define FD_SMALL_SWITCH(NAME, THREADS)         \
  switch (Pl.MD) {                    \
    FD_SMALL_CASE(NAME, THREADS, 1)            \
    FD_SMALL_CASE(NAME, THREADS, 2)            \
    FD_SMALL_CASE(NAME, THREADS, 3)            \
    FD_SMALL_CASE(NAME, THREADS, 4)            \
    FD_SMALL_CASE(NAME, THREADS, 5)            \
    FD_SMALL_CASE(NAME, THREADS, 6)            \
    FD_SMALL_CASE(NAME, THREADS, 7)            \
    FD_SMALL_CASE(NAME, THREADS, 8)            \
    default:                          \
      return hipErrorInvalidValue;    \
  }

template <typename R>
hipError_t launch_point_small_fwd(const Plan& Pl, const DevPlan& P, bool odd, const cx<R>* A, const cx<R>* b,
                                  const cx<R>* c, cx<R>* Ai, void* const* fam, bool ring, cx<R>* rho, hipStream_t st) {
  SmallFwd<R> a;
  std::memset(&a, 0, sizeof(a));
  for (int f = 0; f < Pl.nfam; ++f) a.fam.f[f] = static_cast<cx<R>*>(fam[f]);
  a.fam.ring = ring ? 1 : 0;
  a.A = A;
  a.b = b;
  a.c = c;
  a.Ai = Ai;
  a.rho = rho;
  a.mt = Pl.d_mtab;
  small_prep(Pl, &a.pa);
  a.status = Pl.d_status;
  a.level_order = Pl.level_cap >= 0 ? 1 : 0;
  const size_t shm = 2 * (kMaxCut + 4) * sizeof(R) + (size_t)4 * pt_table_entries(Pl.MD) * 8 +
                     small_tail_lds(Pl, kSmallFwdWaves);
  const bool by_b = odd && Pl.flags == FD_B_AUTO;   // (odd: not known to be zero)
  FD_SMALL_SWITCH(k_point_small_fwd, kSmallFwdThreads)
  return hipGetLastError();
}

template <typename R>
hipError_t launch_point_small_vjp(const Plan& Pl, const DevPlan& P, bool odd, const cx<R>* A, const cx<R>* b,
                                  const cx<R>* c, cx<R>* Ai, void* const* fam, void* const* gfam, const cx<R>* drho,
                                  cx<R>* g0, cx<R>* dA, cx<R>* db, cx<R>* dc, int hi, int lo, double* state,
                                  hipStream_t st) {
  SmallVjp<R> a;
  std::memset(&a, 0, sizeof(a));
  for (int f = 0; f < Pl.nfam; ++f) {
    a.fam.f[f] = static_cast<cx<R>*>(fam[f]);
    a.gfam.f[f] = static_cast<cx<R>*>(gfam[f]);
  }
  a.gfam.ring = 1;
  a.A = A;
  a.b = b;
  a.c = c;
  a.drho = drho;
  a.Ai = Ai;
  a.g0 = g0;
  a.dA = dA;
  a.db = db;
  a.dc = dc;
  a.mt = Pl.d_mtab;
  small_prep(Pl, &a.pa);
  for (int u = 0; u < 2 * kMaxModes; ++u) a.blk2pos[u] = -1;
  for (int p = 0; p < Pl.npos; ++p) a.blk2pos[Pl.pos2blk[p]] = p;
  a.status = Pl.d_status;
  a.level_order = Pl.level_cap >= 0 ? 1 : 0;
  a.hi = hi;
  a.lo = lo;
  a.state = state;
  const size_t shm = std::max(2 * (kMaxCut + 4) * sizeof(R) + (size_t)2 * pt_vjp_entries(Pl.MD) * 8 +
                                  (size_t)kSmallWaves * kPtPos * kTurn * sizeof(cx<R>) + small_tail_lds(Pl, kSmallWaves),
                              (size_t)kSmallWaves * 2 * Pl.MD * (2 * Pl.MD + 1) * sizeof(cx<double>));
  const bool by_b = odd && Pl.flags == FD_B_AUTO && hi == Pl.smax && lo == 0;
  FD_SMALL_SWITCH(k_point_small_vjp, kSmallThreads)
  return hipGetLastError();
}

#define FD_INSTANTIATE(R)                                                                                            \
  template hipError_t launch_point_small_fwd<R>(const Plan&, const DevPlan&, bool, const cx<R>*, const cx<R>*,       \
                                                const cx<R>*, cx<R>*, void* const*, bool, cx<R>*, hipStream_t);      \
  template hipError_t launch_point_small_vjp<R>(const Plan&, const DevPlan&, bool, const cx<R>*, const cx<R>*,       \
                                                const cx<R>*, cx<R>*, void* const*, void* const*, const cx<R>*,      \
                                                cx<R>*, cx<R>*, cx<R>*, cx<R>*, int, int, double*, hipStream_t);
FD_INSTANTIATE(float)
FD_INSTANTIATE(double)

}  // namespace fd
