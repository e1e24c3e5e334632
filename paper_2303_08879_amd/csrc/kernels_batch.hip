// Batched forward: prep and permutation kernels of a batch and the host-side
// schedule (work items, per-circuit descriptors), cached per plan set and
// pointer set.  The level kernels are in kernels_batch_level.hip.
//
// Launch sequence per batch: prep (+ undetected block fill), one workgroup
// per circuit; one launch per class and step, the classes on side streams
// next to the level launches of the circuits that fill the device; the
// F0 -> rho permutation of every circuit in one launch.
#include <algorithm>
#include <cstring>
#include <memory>
#include <mutex>
#include <numeric>

#include "batch_level.h"
#include "pt_units.h"

namespace fd {

// Prep of every circuit (one workgroup each), then step 1 of Algorithm 2 by
// the first wavefront when the circuit has undetected modes.
template <typename R>
__global__ __launch_bounds__(kThreads) void k_batch_prep(const BatchCirc<R>* __restrict__ circs) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const BatchCirc<R>* __restrict__ C = circs + blockIdx.x;
  cx<R>* Ai = load_global(&C->Ai);
  cx<R>* f0 = load_global(&C->f0);
  const int npos = C->P.npos;
  prep_body<R>(load_global(&C->A), load_global(&C->b), load_global(&C->c), Ai, Ai + npos * npos,
               Ai + npos * npos + npos, f0, C->pa, load_global(&C->status));
  if (C->P.B == 1) return;
  __syncthreads();
  if (threadIdx.x < 64) {
    if (C->P.nq == 2)
      ufill_rows_body<R, cx<R>>(C->P, Ai, Ai + npos * npos, f0);
    else
      ufill_body<R, 4>(C->P, Ai, Ai + npos * npos, f0, load_global(&C->elist), load_global(&C->woff), C->wmax,
                       reinterpret_cast<cx<R>*>(smem_raw));
  }
}

// F0 -> rho of every circuit; block b belongs to the circuit c with
// boff[c] <= b < boff[c + 1] and is one LDS tile of it (undetected modes) or
// kThreads x kOutIter consecutive outputs (every mode detected).
template <typename R>
__global__ __launch_bounds__(kThreads) void k_batch_out(const BatchCirc<R>* __restrict__ circs,
                                                        const int64_t* __restrict__ boff, int n, int pn_bytes,
                                                        int slv_bytes) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int64_t blk = blockIdx.x;
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (boff[mid] <= blk)
      lo = mid;
    else
      hi = mid - 1;
  }
  const BatchCirc<R>* __restrict__ C = circs + lo;
  int* spn = reinterpret_cast<int*>(smem_raw);
  int64_t* slv = reinterpret_cast<int64_t*>(smem_raw + pn_bytes);
  const int npn = (C->P.MD + 1) * C->P.pnw;
  const int* pn = load_global(&C->P.pn);
  const int64_t* lvl = load_global(&C->P.lvl);
  for (int i = threadIdx.x; i < npn; i += blockDim.x) spn[i] = pn[i];
  for (int i = threadIdx.x; i <= C->P.smax; i += blockDim.x) slv[i] = C->P.MD > 0 ? lvl[i] : 0;
  __syncthreads();
  const cx<R>* f0 = load_global(&C->f0);
  cx<R>* rho = load_global(&C->rho);
  if (C->P.B > 1) {
    cx<R>* tl = reinterpret_cast<cx<R>*>(smem_raw + pn_bytes + slv_bytes);
    if (out_perm_tile<R>(C->P, spn, slv, f0, rho, C->N, blk - boff[lo], tl)) atomicOr(load_global(&C->status), 1);
    return;
  }
  const int64_t base = (blk - boff[lo]) * (int64_t)kThreads * kOutIter;
  int bad = 0;
#pragma unroll
  for (int k = 0; k < kOutIter; ++k) {
    const int64_t idx = base + (int64_t)k * kThreads + threadIdx.x;
    if (idx < C->out_elems) {
      const cx<R> v = out_perm_elem<R>(C->P, spn, slv, f0, C->N, idx);
      if (!isfinite(v.x) || !isfinite(v.y)) bad = 1;
      st(rho + idx, v);
    }
  }
  if (bad) atomicOr(load_global(&C->status), 1);
}

// ---------------------------------------------------------------------------
// host side: schedule construction (cached per plan set and pointer set)
// ---------------------------------------------------------------------------
namespace {

// The circuits of one kernel instantiation and their launches, one per step.
struct BatchClass {
  int kind = 0, MD = 0, nq = 0, odd = 0;
  std::vector<int> members;
  double work = 0.0;
  struct Step {
    int i0 = 0, n = 0;                 // its items
    size_t shm = 0;
  };
  std::vector<Step> steps;
  int lane = 0;                        // stream it runs on
};

struct BatchSched {
  uint64_t id = 0;                      // unique per built schedule
  bool pinned = false;                  // a caller's captured graph reads its tables: kept as long as the plans
  int device = -1;
  std::vector<uint64_t> key;
  std::vector<uint64_t> uids;
  void* d_circs = nullptr;
  void* d_items = nullptr;
  void* d_boff = nullptr;
  std::vector<BatchClass> classes;     // largest work first
  int64_t out_blocks = 0;
  size_t shm_prep = 0, shm_out = 0;
  int out_pn_bytes = 0, out_slv_bytes = 0;
  uint64_t last_use = 0;
  std::vector<unsigned char> h_circs;   // host images kept alive for the asynchronous uploads
  std::vector<BatchItem> h_items;
  std::vector<int64_t> h_boff;
};

std::mutex g_mu;
std::vector<BatchSched> g_cache;
fd_batch_tuning g_tuning = {2, 64, 4, 2048, 0};

fd_batch_tuning batch_tuning() { return g_tuning; }
// Side streams of a batched call (with the caller's, one per hardware queue; 1 / 2 /
// 3 / 4 streams: 48 uneven circuits 3865 / 2971 / 2943 / 2952 us, 16 of them 1746 /
// 1265 / 1042 / 1049, 8 of them 1603 / 1134 / 800 / 941), and about the workgroups that
// the device holds at once (512 and 8192 take the same time: few steps have more items)
constexpr int kBatchLanes = 3;
constexpr int64_t kBatchResident = 2048;

// Whether the batched level kernels run this circuit: at most four block
// coordinates (two undetected modes), rows and fill staged in LDS.  Others take
// their own level launches.
bool level_launch_takes(const Plan& Pl) {
  return Pl.B == 1 || (Pl.nq <= 4 && !Pl.st_fwd && !Pl.st_ufill);
}
uint64_t g_clock = 0, g_sched_id = 0;
constexpr size_t kBatchCache = 8;

void free_sched(BatchSched& s) {
  if (unloading()) return;   // the HIP runtime may be gone
  int cur = 0;
  (void)hipGetDevice(&cur);
  (void)hipSetDevice(s.device);
  (void)hipFree(s.d_circs);
  (void)hipFree(s.d_items);
  (void)hipFree(s.d_boff);
  (void)hipSetDevice(cur);
  s.d_circs = s.d_items = s.d_boff = nullptr;
}

size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

template <typename R>
fd_status build_sched(int n, Plan* const* plans, const bool* odd, const void* const* A, const void* const* b,
                 const void* const* c, void* const* rho, void* const* ws, hipStream_t st, BatchSched* S,
                 std::string* err) {
  const size_t eb = sizeof(cx<R>);
  std::vector<BatchCirc<R>> hc(n);
  int out_pn = 16;
  int64_t out_slv = 8;
  size_t ufill_lds = 0;
  for (int i = 0; i < n; ++i) {
    const Plan& Pl = *plans[i];
    BatchCirc<R>& C = hc[i];
    std::memset(&C, 0, sizeof(C));
    C.P = make_devplan(Pl, odd[i]);
    if (!level_launch_takes(Pl)) {
      *err = "internal error: a circuit that the batched level kernels do not take";
      return FD_ERR_UNSUPPORTED;
    }
    for (int p = 0; p < Pl.npos; ++p) C.pa.pos2blk[p] = Pl.pos2blk[p];
    C.pa.npos = Pl.npos;
    C.pa.M2 = 2 * Pl.M;
    C.pa.check_b_zero = Pl.flags == FD_B_ZERO ? 1 : 0;
    C.wmax = Pl.wmax;
    const FwdLayout Lw = fwd_layout(Pl, odd[i], false, 0);
    char* w = static_cast<char*>(ws[i]);
    for (int f = 1; f < Pl.nfam; ++f) {
      if (Lw.fam[f] == 0) continue;
      C.fam[f] = reinterpret_cast<cx<R>*>(w + Lw.fam[f]);
      C.fstride[f] = Pl.maxN[Pl.fam_group[f]] * (int64_t)Pl.B;
    }
    C.f0 = reinterpret_cast<cx<R>*>(w + Lw.f0);
    C.Ai = reinterpret_cast<cx<R>*>(w + Lw.prep);
    C.A = static_cast<const cx<R>*>(A[i]);
    C.b = static_cast<const cx<R>*>(b[i]);
    C.c = static_cast<const cx<R>*>(c[i]);
    C.rho = static_cast<cx<R>*>(rho[i]);
    C.mtab = Pl.d_mtab;
    C.elist = Pl.d_elist;
    C.woff = Pl.d_woff;
    C.status = Pl.d_status;
    C.out_elems = Pl.out_elems;
    C.N = Pl.nodes_total;
    const int pnb = (int)align16((size_t)(Pl.MD + 1) * (Pl.smax + 3) * sizeof(int));
    out_pn = std::max(out_pn, pnb);
    out_slv = std::max<int64_t>(out_slv, (int64_t)(Pl.smax + 2) * 8);
    if (Pl.nq > 2) ufill_lds = std::max(ufill_lds, ufill_lds_bytes(Pl, false));
    if (Pl.MD == 0) continue;
    double work = 0.0;
    for (int s = 0; s <= Pl.smax; ++s) work += (double)Pl.ncnt[s] * Pl.B * Pl.npos * Pl.npos;
    const int kind = Pl.B > 1 ? 1 : 0, nq = kind ? Pl.nq : 0, od = kind ? 1 : (odd[i] ? 1 : 0);
    auto it = std::find_if(S->classes.begin(), S->classes.end(), [&](const BatchClass& k) {
      return k.kind == kind && k.MD == Pl.MD && k.nq == nq && k.odd == od;
    });
    if (it == S->classes.end()) {
      BatchClass k;
      k.kind = kind;
      k.MD = Pl.MD;
      k.nq = nq;
      k.odd = od;
      S->classes.push_back(k);
      it = S->classes.end() - 1;
    }
    it->members.push_back(i);
    it->work += work;
  }
  S->shm_prep = ufill_lds;
  S->out_pn_bytes = out_pn;
  S->out_slv_bytes = (int)align16((size_t)out_slv);
  S->shm_out = (size_t)out_pn + S->out_slv_bytes + (size_t)kOutTN * (kOutTK + 1) * eb;

  if (S->shm_prep > 65536 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(&k_batch_prep<R>), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)S->shm_prep) != hipSuccess) {
    *err = "hipFuncSetAttribute failed";
    return FD_ERR_HIP;
  }
  int dev = 0;
  (void)hipGetDevice(&dev);
  // work items: every step of a circuit in workgroups of whole units, one
  // (lattice point, chunk) unit or one 16-column pass each unless the
  // step has more than items_per_wave x kBatchResident of them
  const fd_batch_tuning T = batch_tuning();
  std::stable_sort(S->classes.begin(), S->classes.end(),
                   [](const BatchClass& x, const BatchClass& y) { return x.work > y.work; });
  S->h_items.clear();
  for (BatchClass& k : S->classes) {
    int max_steps = 0;
    for (int i : k.members) max_steps = std::max(max_steps, plans[i]->smax + 1);
    k.steps.assign(max_steps, BatchClass::Step());
    for (int s = 0; s < max_steps; ++s) {
      BatchClass::Step& st_ = k.steps[s];
      st_.i0 = (int)S->h_items.size();
      for (int i : k.members) {
        const Plan& Pl = *plans[i];
        if (s > Pl.smax || Pl.ncnt[s] <= 0) continue;
        const int64_t pts = Pl.ncnt[s];
        BatchItem I;
        std::memset(&I, 0, sizeof(I));
        I.circ = i;
        int64_t units = pts, per;
        if (k.kind) {
          const ChunkGeo G = fwd_geo(Pl, pts);
          I.RC = G.RC;
          I.nchunks = G.nchunks;
          units = pts * G.nchunks;
          per = std::max<int64_t>((T.min_block_units + 1) / 2, units / ((int64_t)T.items_per_wave * kBatchResident));
          st_.shm = std::max(st_.shm, fwd_lds_bytes_for(Pl, G));
        } else {
          const PtItems N = pt_items(Pl, s);
          units = 0;
          for (int K = 0; K < Pl.MD; ++K) units += N.tiles(K);
          // min_point_units counts lattice points, 16 per item
          per = std::max<int64_t>({kThreads / 64, T.min_point_units / 16,
                                   units / ((int64_t)T.items_per_wave * kBatchResident)});
          st_.shm = std::max(st_.shm, pt_lds_bytes(Pl, 1, kThreads / 64, 2));
        }
        if (units > 0x7fffffff) {
          *err = "a step of circuit " + std::to_string(i) + " has too many units for one work item table";
          return FD_ERR_UNSUPPORTED;
        }
        if ((k.kind && (I.RC < 1 || I.nchunks < 1 || (int64_t)(I.nchunks - 1) * I.RC >= Pl.udims[0])) ||
            !batch_cut(units, per, I, &S->h_items)) {
          *err = "internal error: a work item of circuit " + std::to_string(i) + " outside its step";
          return FD_ERR_UNSUPPORTED;
        }
      }
      st_.n = (int)S->h_items.size() - st_.i0;
    }
  }
  // streams: largest class first, each to the stream with the least work
  double load[kBatchLanes] = {};
  for (BatchClass& k : S->classes) {
    k.lane = (int)(std::min_element(load, load + kBatchLanes) - load);
    load[k.lane] += k.work;
  }
  // permutation blocks
  S->h_boff.assign(n + 1, 0);
  for (int i = 0; i < n; ++i) {
    const int64_t per_blk = (int64_t)kThreads * kOutIter;
    const int64_t blocks = hc[i].P.B > 1 ? ((hc[i].N + kOutTN - 1) / kOutTN) * ((hc[i].P.B + kOutTK - 1) / kOutTK)
                                         : (hc[i].out_elems + per_blk - 1) / per_blk;
    S->h_boff[i + 1] = S->h_boff[i] + blocks;
  }
  S->out_blocks = S->h_boff[n];
  if (S->out_blocks > 0x7fffffff) {
    *err = "batch output too large for one permutation launch";
    return FD_ERR_UNSUPPORTED;
  }
  // upload
  S->h_circs.resize(sizeof(BatchCirc<R>) * n);
  std::memcpy(S->h_circs.data(), hc.data(), S->h_circs.size());
  S->device = dev;
  if (hipMalloc(&S->d_circs, S->h_circs.size()) != hipSuccess ||
      hipMalloc(&S->d_items, std::max<size_t>(1, S->h_items.size()) * sizeof(BatchItem)) != hipSuccess ||
      hipMalloc(&S->d_boff, S->h_boff.size() * sizeof(int64_t)) != hipSuccess) {
    free_sched(*S);
    *err = "device allocation of the batch schedule failed";
    return FD_ERR_OOM;
  }
  if (hipMemcpyAsync(S->d_circs, S->h_circs.data(), S->h_circs.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
      (!S->h_items.empty() && hipMemcpyAsync(S->d_items, S->h_items.data(), S->h_items.size() * sizeof(BatchItem),
                                       hipMemcpyHostToDevice, st) != hipSuccess) ||
      hipMemcpyAsync(S->d_boff, S->h_boff.data(), S->h_boff.size() * sizeof(int64_t), hipMemcpyHostToDevice,
                     st) != hipSuccess) {
    free_sched(*S);
    *err = "upload of the batch schedule failed";
    return FD_ERR_HIP;
  }
  return FD_OK;
}

// Side streams of a batched call and the events that order them after the
// caller's stream and it after them, per device, kept until the process ends.
// Used under g_mu; a call that finds earlier work on a side stream queues
// behind it.
struct BatchLanes {
  hipStream_t s[kBatchLanes] = {};
  hipEvent_t fork = nullptr, join[kBatchLanes] = {};
};
BatchLanes g_lanes[64];

hipError_t batch_lanes(int dev, BatchLanes** out) {
  BatchLanes& L = g_lanes[dev];
  hipError_t e = hipSuccess;
  if (!L.fork) e = hipEventCreateWithFlags(&L.fork, hipEventDisableTiming);
  for (int k = 0; k < kBatchLanes && e == hipSuccess; ++k) {
    if (!L.s[k]) e = hipStreamCreateWithFlags(&L.s[k], hipStreamNonBlocking);
    if (e == hipSuccess && !L.join[k]) e = hipEventCreateWithFlags(&L.join[k], hipEventDisableTiming);
  }
  *out = &L;
  return e;
}

// The steps of the classes of one stream, class by class.
template <typename R>
hipError_t launch_lane(const BatchSched& S, int lane, hipStream_t st) {
  for (const BatchClass& k : S.classes) {
    if (k.lane != lane) continue;
    for (size_t s = 0; s < k.steps.size(); ++s) {
      if (k.steps[s].n == 0) continue;
      BatchLaunch a{};
      a.kind = k.kind;
      a.MD = k.MD;
      a.nq = k.nq;
      a.odd = k.odd;
      a.circs = S.d_circs;
      a.items = static_cast<const BatchItem*>(S.d_items) + k.steps[s].i0;
      a.nitems = k.steps[s].n;
      a.S = (int)s;
      a.shm = k.steps[s].shm;
      const hipError_t e = launch_batch_level<R>(a, st);
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

template <typename R>
hipError_t launch_batch_prep(const BatchSched& S, int n, const Plan& P0, hipStream_t st) {
  KTimer kt(P0, KK_BATCH_PREP, st);
  hipLaunchKernelGGL((k_batch_prep<R>), dim3(n), dim3(kThreads), S.shm_prep, st,
                     static_cast<const BatchCirc<R>*>(S.d_circs));
  return hipGetLastError();
}

template <typename R>
hipError_t launch_batch_out(const BatchSched& S, int n, const Plan& P0, hipStream_t st) {
  KTimer kt(P0, KK_BATCH_OUT, st);
  hipLaunchKernelGGL((k_batch_out<R>), dim3((unsigned)S.out_blocks), dim3(kThreads), S.shm_out, st,
                     static_cast<const BatchCirc<R>*>(S.d_circs), static_cast<const int64_t*>(S.d_boff), n,
                     S.out_pn_bytes, S.out_slv_bytes);
  return hipGetLastError();
}

}  // namespace

// A circuit fills the device on its own when its levels average at least
// `fill_waves` wavefront-sized units (about what the device holds at once,
// 2048 by default): such circuits run their own level launches, interleaving
// them with other large circuits only multiplies the working set the L2s and
// the MALL hold.
static bool fills_device(const Plan& Pl, double fill_waves) {
  if (Pl.MD == 0) return false;
  double units = 0.0;
  const ChunkGeo G = Pl.B > 1 ? chunk_geo(Pl) : ChunkGeo{1, 1, 1, 1};
  for (int s = 0; s <= Pl.smax; ++s)
    units += Pl.B > 1 ? (double)Pl.ncnt[s] * G.nchunks : (double)Pl.ncnt[s] / 64.0;
  return units / (Pl.smax + 1) >= fill_waves;
}

namespace {

// A batched call captured into a graph.
struct BatchGraph {
  int device = -1;
  uint64_t sched = 0;                // schedule whose device tables the graph's kernels read (0: none)
  std::vector<uint64_t> key, uids;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  uint64_t last_use = 0;
};
std::vector<BatchGraph> g_graphs;
hipStream_t g_capture[64] = {};   // private capture stream per device
bool g_graph_failed = false;      // a capture was refused: batched calls run eagerly

void free_graph(BatchGraph& g) {
  if (unloading()) return;
  (void)hipGraphExecDestroy(g.exec);
  (void)hipGraphDestroy(g.graph);
  g.exec = nullptr;
  g.graph = nullptr;
}

// Drops a schedule and every graph captured over its device tables: a graph
// replayed after its schedule was evicted would read freed memory.
void drop_sched(BatchSched& s) {
  for (size_t i = 0; i < g_graphs.size();) {
    if (g_graphs[i].sched == s.id) {
      free_graph(g_graphs[i]);
      g_graphs.erase(g_graphs.begin() + i);
    } else {
      ++i;
    }
  }
  free_sched(s);
}

// Cache key of a batched call: device, plans, schedules, pointers, knobs.
std::vector<uint64_t> batch_key(int n, Plan* const* plans, const bool* odd, const void* const* A,
                                const void* const* b, const void* const* c, void* const* rho, void* const* ws,
                                const fd_batch_tuning& T) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::vector<uint64_t> key;
  key.reserve(7 + 7 * (size_t)n);
  key.push_back((uint64_t)dev);
  key.push_back((uint64_t)n);
  for (int i = 0; i < n; ++i) {
    key.push_back(plans[i]->uid);
    key.push_back(odd[i] ? 1 : 0);
    for (const void* p : {A[i], b[i], c[i], (const void*)rho[i], (const void*)ws[i]})
      key.push_back((uint64_t)reinterpret_cast<uintptr_t>(p));
  }
  key.push_back((uint64_t)T.min_block_units);
  key.push_back((uint64_t)T.min_point_units);
  key.push_back((uint64_t)T.items_per_wave);
  key.push_back((uint64_t)T.fill_waves);
  return key;
}

// The schedule of the level launches over these circuits, built and
// uploaded on `st` on first use.  Caller holds g_mu.
fd_status sweep_sched(int n, Plan* const* plans, const bool* odd, const void* const* A, const void* const* b,
                      const void* const* c, void* const* rho, void* const* ws, const fd_batch_tuning& T,
                      hipStream_t st, BatchSched** out, std::string* err) {
  std::vector<uint64_t> key = batch_key(n, plans, odd, A, b, c, rho, ws, T);
  for (BatchSched& s : g_cache)
    if (s.key == key) {
      s.last_use = ++g_clock;
      *out = &s;
      return FD_OK;
    }
  BatchSched ns;
  ns.key = std::move(key);
  for (int i = 0; i < n; ++i) ns.uids.push_back(plans[i]->uid);
  const fd_status bs = plans[0]->dt == FD_C64 ? build_sched<float>(n, plans, odd, A, b, c, rho, ws, st, &ns, err)
                                              : build_sched<double>(n, plans, odd, A, b, c, rho, ws, st, &ns, err);
  if (bs != FD_OK) return bs;
  if (std::count_if(g_cache.begin(), g_cache.end(), [](const BatchSched& x) { return !x.pinned; }) >=
      (std::ptrdiff_t)kBatchCache) {
    auto it = std::min_element(g_cache.begin(), g_cache.end(), [](const BatchSched& x, const BatchSched& y) {
      return x.pinned != y.pinned ? y.pinned : x.last_use < y.last_use;
    });
    drop_sched(*it);
    g_cache.erase(it);
  }
  ns.id = ++g_sched_id;
  g_cache.push_back(std::move(ns));
  *out = &g_cache.back();
  (*out)->last_use = ++g_clock;
  return FD_OK;
}

struct Split {
  std::vector<int> big, small;
};

Split split_batch(int n, Plan* const* plans, const fd_batch_tuning& T) {
  Split sp;
  for (int i = 0; i < n; ++i)
    (fills_device(*plans[i], (double)T.fill_waves) || !level_launch_takes(*plans[i]) ? sp.big : sp.small).push_back(i);
  return sp;
}

// Enqueues the whole batched call on `st`: prep of the batched circuits, then
// their classes on the side streams while `st` runs the level launches of the
// circuits that fill the device (or that the batched kernels do not take), then
// the permutation.  `st` waits for the side streams before it goes on, so
// everything the call touches is ordered on `st`.  Without `fork` everything
// runs on `st`: a stream that the caller captures would draw the side streams into
// its capture, and every other batched call that then used them would fail.
template <typename R>
hipError_t enqueue_batch_t(const Split& sp, Plan* const* plans, const bool* odd, const void* const* A,
                           const void* const* b, const void* const* c, void* const* rho, void* const* ws,
                           const BatchSched* S, bool fork, hipStream_t st) {
  hipError_t e = hipSuccess;
  auto big = [&]() -> hipError_t {
    for (int i : sp.big) {
      const hipError_t x = run_forward(*plans[i], odd[i], A[i], b[i], c[i], rho[i], ws[i], nullptr, st);
      if (x != hipSuccess) return x;
    }
    return hipSuccess;
  };
  if (!S) return big();
  const int n = (int)sp.small.size();
  const Plan& P0 = *plans[sp.small[0]];
  if ((e = launch_batch_prep<R>(*S, n, P0, st)) != hipSuccess) return e;
  if (!fork) {
    {
      KTimer kt(P0, KK_BATCH_SWEEP, st);
      if ((e = big()) != hipSuccess) return e;
      for (int k = 0; k < kBatchLanes; ++k)
        if ((e = launch_lane<R>(*S, k, st)) != hipSuccess) return e;
    }
    return launch_batch_out<R>(*S, n, P0, st);
  }
  BatchLanes* L = nullptr;
  if ((e = batch_lanes(S->device, &L)) != hipSuccess) return e;
  bool used[kBatchLanes] = {};
  for (const BatchClass& k : S->classes) used[k.lane] = true;
  {
    KTimer kt(P0, KK_BATCH_SWEEP, st);
    if ((e = hipEventRecord(L->fork, st)) != hipSuccess) return e;
    hipError_t bad = hipSuccess;
    for (int k = 0; k < kBatchLanes; ++k)
      if (used[k] && bad == hipSuccess) bad = hipStreamWaitEvent(L->s[k], L->fork, 0);
      else used[k] = false;
    // the large circuits first: the device works on them while the host
    // enqueues the others
    if (bad == hipSuccess) bad = big();
    for (int k = 0; k < kBatchLanes; ++k)
      if (used[k] && bad == hipSuccess) bad = launch_lane<R>(*S, k, L->s[k]);
    // every stream that was forked is joined, also after an error
    for (int k = 0; k < kBatchLanes; ++k)
      if (used[k]) {
        e = hipEventRecord(L->join[k], L->s[k]);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, L->join[k], 0);
        if (bad == hipSuccess) bad = e;
      }
    if (bad != hipSuccess) return bad;
  }
  return launch_batch_out<R>(*S, n, P0, st);
}

hipError_t enqueue_batch(const Split& sp, Plan* const* plans, const bool* odd, const void* const* A,
                         const void* const* b, const void* const* c, void* const* rho, void* const* ws,
                         const BatchSched* S, bool fork, hipStream_t st) {
  const bool c64 = !sp.small.empty() && plans[sp.small[0]]->dt == FD_C64;
  return c64 ? enqueue_batch_t<float>(sp, plans, odd, A, b, c, rho, ws, S, fork, st)
             : enqueue_batch_t<double>(sp, plans, odd, A, b, c, rho, ws, S, fork, st);
}

}  // namespace

fd_status run_forward_batch(int n, Plan* const* plans, const bool* odd, const void* const* A,
                            const void* const* b, const void* const* c, void* const* rho, void* const* ws,
                            hipStream_t st, std::string* err) {
  if (n == 0) return FD_OK;
  std::lock_guard<std::mutex> lock(g_mu);
  const fd_batch_tuning T = g_tuning;
  const Split sp = split_batch(n, plans, T);
  // the batched members, as arrays of their own
  const size_t m = sp.small.size();
  std::vector<Plan*> p2(m);
  std::unique_ptr<bool[]> o2(new bool[m > 0 ? m : 1]);
  std::vector<const void*> A2(m), b2(m), c2(m);
  std::vector<void*> r2(m), w2(m);
  for (size_t k = 0; k < m; ++k) {
    const int i = sp.small[k];
    p2[k] = plans[i];
    o2[k] = odd[i];
    A2[k] = A[i];
    b2[k] = b[i];
    c2[k] = c[i];
    r2[k] = rho[i];
    w2[k] = ws[i];
  }
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();   // not left for the launches' checks
  const bool captured_by_caller = cap != hipStreamCaptureStatusNone;
  auto fail_hip = [&](hipError_t e) {
    *err = std::string("kernel launch failed: ") + hipGetErrorString(e);
    return FD_ERR_HIP;
  };
  int dev = 0;
  (void)hipGetDevice(&dev);
  if (dev < 0 || dev >= 64) return fail_hip(hipErrorInvalidDevice);
  BatchSched* S = nullptr;
  if (m > 0) {
    // an upload captured by the caller would not have run when the next call
    // finds the schedule: it goes to a side stream and is waited for
    hipStream_t up = st;
    BatchLanes* L = nullptr;
    if (captured_by_caller) {
      const hipError_t e = batch_lanes(dev, &L);
      if (e != hipSuccess) return fail_hip(e);
      up = L->s[0];
    }
    const uint64_t built = g_sched_id;
    const fd_status s = sweep_sched((int)m, p2.data(), o2.get(), A2.data(), b2.data(), c2.data(), r2.data(),
                                    w2.data(), T, up, &S, err);
    if (s != FD_OK) return s;
    if (captured_by_caller && g_sched_id != built) {
      const hipError_t e = hipStreamSynchronize(up);
      if (e != hipSuccess) return fail_hip(e);
    }
    S->pinned = S->pinned || captured_by_caller;
  }
  bool timing = false;
  for (int i = 0; i < n; ++i) timing = timing || plans[i]->timing.mask != 0;
  if (T.use_graph <= 0 || g_graph_failed || timing) {
    const hipError_t e = enqueue_batch(sp, plans, odd, A, b, c, rho, ws, S, !captured_by_caller, st);
    return e == hipSuccess ? FD_OK : fail_hip(e);
  }
  std::vector<uint64_t> key = batch_key(n, plans, odd, A, b, c, rho, ws, T);
  for (BatchGraph& g : g_graphs)
    if (g.key == key) {
      g.last_use = ++g_clock;
      const hipError_t e = hipGraphLaunch(g.exec, st);
      return e == hipSuccess ? FD_OK : fail_hip(e);
    }
  hipError_t e;
  if (!g_capture[dev] && (e = hipStreamCreateWithFlags(&g_capture[dev], hipStreamNonBlocking)) != hipSuccess)
    return fail_hip(e);
  hipStream_t cs = g_capture[dev];
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  bool captured = false;
  if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) == hipSuccess) {
    const hipError_t eb = enqueue_batch(sp, plans, odd, A, b, c, rho, ws, S, true, cs);
    const hipError_t ee = hipStreamEndCapture(cs, &graph);
    captured = eb == hipSuccess && ee == hipSuccess && graph &&
               hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) == hipSuccess;
  }
  (void)hipGetLastError();
  if (!captured) {
    // the runtime would not capture: run this and later calls eagerly
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    g_graph_failed = true;
    e = enqueue_batch(sp, plans, odd, A, b, c, rho, ws, S, !captured_by_caller, st);
    return e == hipSuccess ? FD_OK : fail_hip(e);
  }
  if (g_graphs.size() >= kBatchCache) {
    auto it = std::min_element(g_graphs.begin(), g_graphs.end(),
                               [](const BatchGraph& x, const BatchGraph& y) { return x.last_use < y.last_use; });
    free_graph(*it);
    g_graphs.erase(it);
  }
  BatchGraph g;
  g.device = dev;
  g.sched = S ? S->id : 0;
  g.key = std::move(key);
  for (int i = 0; i < n; ++i) g.uids.push_back(plans[i]->uid);
  g.graph = graph;
  g.exec = exec;
  g.last_use = ++g_clock;
  g_graphs.push_back(std::move(g));
  e = hipGraphLaunch(exec, st);
  return e == hipSuccess ? FD_OK : fail_hip(e);
}

fd_status batch_set_tuning(const fd_batch_tuning& T) {
  if (T.min_block_units < 1 || T.min_point_units < 1 || T.items_per_wave < 1 || T.fill_waves < 1 ||
      T.use_graph < 0 || T.use_graph > 1)
    return FD_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lock(g_mu);
  g_tuning = T;
  return FD_OK;
}

fd_batch_tuning batch_get_tuning() {
  std::lock_guard<std::mutex> lock(g_mu);
  fd_batch_tuning t = g_tuning;
  if (t.use_graph > 0 && g_graph_failed) t.use_graph = -1;
  return t;
}

void batch_forget(uint64_t uid) {
  std::lock_guard<std::mutex> lock(g_mu);
  for (size_t i = 0; i < g_graphs.size();) {
    if (std::find(g_graphs[i].uids.begin(), g_graphs[i].uids.end(), uid) != g_graphs[i].uids.end()) {
      free_graph(g_graphs[i]);
      g_graphs.erase(g_graphs.begin() + i);
    } else {
      ++i;
    }
  }
  for (size_t i = 0; i < g_cache.size();) {
    if (std::find(g_cache[i].uids.begin(), g_cache[i].uids.end(), uid) != g_cache[i].uids.end()) {
      drop_sched(g_cache[i]);
      g_cache.erase(g_cache.begin() + i);
    } else {
      ++i;
    }
  }
}

}  // namespace fd
