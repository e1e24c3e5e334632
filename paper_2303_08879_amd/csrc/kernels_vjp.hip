// Reverse sweep (vector-Jacobian product) of the selective recurrence.
//
// Forward, every computed amplitude t has one canonical parent pivot p and
// direction i:  G_t = (b_i G_p + sum_l sqrt(p_l) A_il G_{p-1_l}) / sqrt(p_i+1)
// (Eq. recrel).  With h_t = gbar_t / sqrt(p_i + 1), the adjoint (Sec. 2.5,
// Eqs. dL_dB / dL_dA, in reverse instead of forward mode) is
//   gbar_{p-1_l} += sqrt(p_l) conj(A_il) h_t,   gbar_p += conj(b_i) h_t,
//   Abar_il      += conj(sqrt(p_l) G_{p-1_l}) h_t,   bbar_i += conj(G_p) h_t.
// The sweep visits the levels of the forward in reverse.  Each off-diagonal
// amplitude is read by exactly one pivot (Sec. 3.1.4 / App. B.2), so the
// cotangent slot of every read is *written* (not accumulated) by the thread
// of its only reader: no atomics, and two-level rings suffice for the
// cotangents.  Diagonal amplitudes F0(m) are read only by pivots that sit at
// the same lattice point m, so their cotangents are summed locally.
// Abar / bbar are sums over every target: products h conj(x)^T on the matrix
// cores, summed in registers; each workgroup adds its wavefronts' sums in order to
// its own partial slot, and one final kernel sums the slots in order.  The result
// is bitwise reproducible for a given plan.  This file: the cotangent permutation,
// the reverse of the block fill, the final sums and the driver (level kernels:
// vjp_point_units.h, vjp_block.h).
#include <algorithm>
#include <cstring>

#include "vjp_common.h"

namespace fd {

template <typename R>
__global__ void k_zero_cx(cx<R>* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    st(p + i, czero<R>());
}

__global__ void k_zero_d2(double2* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = make_double2(0.0, 0.0);
}

// rho-shaped cotangent (C order [kappa][n_D]) -> node order (level-major)
template <typename R, int EPT>
__global__ __launch_bounds__(kThreads) void k_perm_in(DevPlan P, const cx<R>* __restrict__ drho, cx<R>* __restrict__ g0,
                                                      int64_t N, int64_t total) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  int* spn = reinterpret_cast<int*>(smem_raw);
  int64_t* slv = reinterpret_cast<int64_t*>(smem_raw + 16 * ((((P.MD + 1) * P.pnw) * 4 + 15) / 16));
  const int npn = (P.MD + 1) * P.pnw;
  for (int i = threadIdx.x; i < npn; i += blockDim.x) spn[i] = P.pn[i];
  for (int i = threadIdx.x; i <= P.smax; i += blockDim.x) slv[i] = P.MD > 0 ? P.lvl[i] : 0;
  __syncthreads();
  const int B = P.B;
  if (B > 1) {
    // tiles of kOutTN consecutive C-order lattice points n by kOutTK block
    // entries kappa through LDS, the inverse of the output permutation: each
    // kappa's run of n is read as one, each node's run of kappa written as one
    cx<R>* tl = reinterpret_cast<cx<R>*>(reinterpret_cast<unsigned char*>(slv) + 16 * (((P.smax + 2) * 8 + 15) / 16));
    constexpr int LD = kOutTK + 1;
    const int64_t ntn = (N + kOutTN - 1) / kOutTN, tiles = ntn * ((B + kOutTK - 1) / kOutTK);
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
      const int64_t n0 = (tile % ntn) * kOutTN;
      const int kap0 = (int)(tile / ntn) * kOutTK;
      {
        const int nl = threadIdx.x % kOutTN;
        for (int k = threadIdx.x / kOutTN; k < kOutTK; k += kThreads / kOutTN)
          if (n0 + nl < N && kap0 + k < B) tl[nl * LD + k] = ld(drho + (size_t)(kap0 + k) * N + n0 + nl);
      }
      __syncthreads();
      const int kl = threadIdx.x % kOutTK, nl0 = threadIdx.x / kOutTK;
      const int node = out_tile_node(P, spn, slv, n0, N);
#pragma unroll
      for (int e = 0; e < kOutTN * kOutTK / kThreads; ++e) {
        const int nl = nl0 + e * (kThreads / kOutTK), nd = __shfl(node, nl);
        if (n0 + nl < N && kap0 + kl < B) st(g0 + (size_t)nd * B + kap0 + kl, tl[nl * LD + kl]);
      }
      __syncthreads();
    }
    return;
  }
  // one entry per node (no undetected modes): C-order index -> node order
  for (int64_t i0 = (int64_t)blockIdx.x * kThreads * EPT; i0 < total;
       i0 += (int64_t)gridDim.x * kThreads * EPT) {
    cx<R> v[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) v[e] = ld(drho + min(i0 + e * kThreads + threadIdx.x, total - 1));
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int64_t idx = i0 + e * kThreads + threadIdx.x;
      if (idx < total) st(g0 + node_of_cindex(P, spn, slv, (int)idx), v[e]);
    }
  }
}

// ---------------------------------------------------------------------------
// Reverse of step 1 of Algorithm 2 (undetected block at zero detections), by
// weight from the top, one wavefront with the block's forward values and
// cotangents in LDS: an entry's cotangent gathers from the targets that used
// it as pivot (x + 1_q with first non-zero coordinate q) or as a read
// (x + 1_q2 + 1_q with parent x + 1_q2, first non-zero coordinate q).
// As in the forward fill, every operand of the weight steps is staged in LDS
// first (incoming cotangents included), so the steps never wait on global
// memory.  LDS: ufill_lds_bytes(plan, true).
// ---------------------------------------------------------------------------
template <typename R, int NQ, bool ST = false>
__global__ __launch_bounds__(64) void k_ufill_vjp(DevPlan P, const cx<R>* __restrict__ Ai,
                                                  const cx<R>* __restrict__ bi, const cx<R>* __restrict__ G,
                                                  const cx<R>* __restrict__ gin, const int* __restrict__ elist,
                                                  const int* __restrict__ woff, int wmax, double2* slot,
                                                  cx<R>* cbar, cx<R>* gbuf) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int nq = NQ;   // 2 per undetected mode
  const int npos = P.npos, B = P.B;
  const int NR = npos + 1;
  const int lane = threadIdx.x;
  // forward values and cotangents of the block: in LDS, or (ST) read from
  // HBM where the forward left them and accumulated in `gbuf` (B entries of
  // the workspace)
  cx<R>* Gl = reinterpret_cast<cx<R>*>(smem_raw);
  cx<R>* gf = ST ? gbuf : Gl + B;
  cx<R>* sA = ST ? Gl : gf + B;   // A between undetected positions, row stride NQ
  cx<R>* sb = sA + NQ * NQ;
  R* sq = reinterpret_cast<R*>(sb + NQ);
  R* isq = sq + (kMaxCut + 4);
  const int* el = elist;
  const int* wo = woff;
  auto GL = [&](int i) -> cx<R> {
    if constexpr (ST)
      return ld(G + i);
    else
      return Gl[i];
  };
  if constexpr (ST) {
    for (int e = lane; e < B; e += 64) st(gf + e, ld(gin + e));
  } else {
    int* lel = reinterpret_cast<int*>(isq + (kMaxCut + 4));
    int* lwo = lel + B;
    for (int e = lane; e < B; e += 64) {
      Gl[e] = ld(G + e);
      gf[e] = ld(gin + e);
      lel[e] = elist[e];
    }
    for (int t = lane; t < wmax + 2; t += 64) lwo[t] = woff[t];
    el = lel;
    wo = lwo;
  }
  for (int i = lane; i < nq * nq; i += 64) sA[(i / nq) * NQ + i % nq] = ld(Ai + (i / nq) * npos + i % nq);
  if (lane < nq) sb[lane] = ld(bi + lane);
  for (int v = lane; v < kMaxCut + 4; v += 64) {
    sq[v] = sqrt(R(v));
    isq[v] = v ? R(1) / sqrt(R(v)) : R(0);
  }
  unit_sync<ST>();
  cx<double> ab[NQ][NQ + 1];
#pragma unroll
  for (int a = 0; a < NQ; ++a)
#pragma unroll
    for (int c = 0; c <= NQ; ++c) ab[a][c] = cmake<double>(0.0, 0.0);
  for (int w = wmax; w >= 0; --w) {
    const int t1 = wo[w + 1];
    for (int t = wo[w] + lane; t < t1; t += 64) {
      const int e = el[t];
      int x[NQ];
      int rem = e;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        x[q] = q < nq ? ucoord(P, rem, q) : 0;
        rem -= x[q] * (q < nq ? P.ustride[q] : 0);
      }
      // first non-zero coordinate, its stride and value, selected with
      // constant indices (a lane-dependent index into the plan's arrays
      // would fetch them from argument memory on every step)
      int first0 = nq, usf = 0, xf = 0;
#pragma unroll
      for (int q = NQ - 1; q >= 0; --q)
        if (q < nq && x[q] > 0) {
          first0 = q;
          usf = P.ustride[q];
          xf = x[q];
        }
      cx<R> acc = gf[e];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (q >= nq || q > first0) continue;
        if (x[q] + 1 < P.udims[q]) {
          const cx<R> ht = cscale(gf[e + P.ustride[q]], isq[x[q] + 1]);
          cfma_conj(acc, sb[q], ht);
        }
#pragma unroll
        for (int q2 = 0; q2 < NQ; ++q2) {
          if (q2 < q || q2 >= nq) continue;
          const int p2 = x[q2] + 1;                  // parent coordinate along q2
          const int pq = x[q] + (q2 == q ? 1 : 0);   // parent coordinate along q
          if (p2 >= P.udims[q2] || pq + 1 >= P.udims[q]) continue;
          const cx<R> ht = cscale(gf[e + P.ustride[q2] + P.ustride[q]], isq[pq + 1]);
          cx<R> u = czero<R>();
          cfma_conj(u, sA[q * NQ + q2], ht);
          acc = cadd(acc, cscale(u, sq[p2]));
        }
      }
      gf[e] = acc;
      if (e > 0) {
        // this entry as a target: parent x - 1_first0, direction first0
        const int qf = first0;
        const int pe = e - usf;
        const cx<R> h = cscale(acc, isq[xf]);
        const cx<R> gp = GL(pe);
#pragma unroll
        for (int a = 0; a < NQ; ++a) {
          if (a != qf) continue;
          ab[a][NQ].x += (double)gp.x * h.x + (double)gp.y * h.y;
          ab[a][NQ].y += (double)gp.x * h.y - (double)gp.y * h.x;
#pragma unroll
          for (int q2 = 0; q2 < NQ; ++q2) {
            if (q2 >= nq) continue;
            const int pq2 = x[q2] - (q2 == qf ? 1 : 0);
            if (pq2 <= 0) continue;
            const cx<R> g2 = cscale(GL(pe - P.ustride[q2]), sq[pq2]);
            ab[a][q2].x += (double)g2.x * h.x + (double)g2.y * h.y;
            ab[a][q2].y += (double)g2.x * h.y - (double)g2.y * h.x;
          }
        }
      }
    }
    unit_sync<ST>();
  }
  // butterfly sums over the wavefront (fixed order), lane 0 adds to the slot
#pragma unroll
  for (int a = 0; a < NQ; ++a) {
#pragma unroll
    for (int c = 0; c <= NQ; ++c) {
      if (a >= nq || (c >= nq && c != NQ)) continue;   // uniform
      double vx = ab[a][c].x, vy = ab[a][c].y;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        vx += __shfl_xor(vx, off, 64);
        vy += __shfl_xor(vy, off, 64);
      }
      if (lane == 0) {
        const int p = a * NR + (c == NQ ? npos : c);
        double2 v = slot[p];
        slot[p] = make_double2(v.x + vx, v.y + vy);
      }
    }
  }
  if (lane == 0) st(cbar, gf[0]);
}

// The same for one undetected mode, row by row from the last (see
// ufill_rows_body): lane l holds column l of the cotangents of three rows.
template <typename R>
__global__ __launch_bounds__(64) void k_ufill_vjp_rows(DevPlan P, const cx<R>* __restrict__ Ai,
                                                       const cx<R>* __restrict__ bi, const cx<R>* __restrict__ G,
                                                       const cx<R>* __restrict__ gin, double2* slot, cx<R>* cbar) {
  const int C = P.udims[0], npos = P.npos, NR = npos + 1, lane = threadIdx.x;
  const R* sqt = reinterpret_cast<const R*>(P.sqt);
  const R sql = sqt[lane], isql = sqt[kMaxCut + 4 + lane], sqr = sqt[lane + 1];
  const cx<R> b0 = ld(bi), b1 = ld(bi + 1), a00 = ld(Ai), a01 = ld(Ai + 1), a11 = ld(Ai + npos + 1);
  const bool in = lane < C;
  const int col = in ? lane : 0;
  auto row = [&](const cx<R>* M, int k) { return csel(in && k >= 0, ld(M + (k >= 0 ? k : 0) * C + col), czero<R>()); };
  // sums h conj(x): rows 0 (direction ket) with x = b term, A00, A01 reads and
  // 1 (direction bra) with b term, A11 read
  double sx[5] = {}, sy[5] = {};
  auto add = [&](int i, const cx<R>& h, const cx<R>& x) {
    const double hx = h.x, hy = h.y, px = x.x, py = x.y;
    sx[i] += px * hx + py * hy;
    sy[i] += px * hy - py * hx;
  };
  // cotangents of rows k, k - 1 (the latter without what row k adds), forward
  // values of rows k - 1, k - 2; the row below next is loaded a step ahead
  cx<R> gk = row(gin, C - 1), g1 = row(gin, C - 2), g2 = row(gin, C - 3);
  cx<R> f1 = row(G, C - 2), f2 = row(G, C - 3), f3 = row(G, C - 4);
  for (int k = C - 1; k >= 1; --k) {
    const cx<R> gn = row(gin, k - 3), fn = row(G, k - 4);
    const cx<R> h = cscale(gk, lane_value(isql, k));
    const R wk = lane_value(sql, k - 1);
    add(0, h, f1);
    add(1, h, cscale(f2, wk));
    const cx<R> fl = shfl_el(f1, lane > 0 ? lane - 1 : 0), hr = shfl_el(h, min(lane + 1, 63));
    add(2, h, cscale(fl, sql));   // weight 0 in lane 0
    cfma_conj(g1, b0, h);
    if (lane + 1 < C) cfma_conj(g1, a01, cscale(hr, sqr));
    cfma_conj(g2, a00, cscale(h, wk));
    gk = g1;
    g1 = g2;
    g2 = gn;
    f1 = f2;
    f2 = f3;
    f3 = fn;
  }
  // row 0: entry l from l - 1 and l - 2
  const cx<R> f0 = row(G, 0);
  cx<R> h0 = czero<R>();                       // lane l: its h
  cx<R> cur = shfl_el(gk, C - 1), nxt = shfl_el(gk, C >= 2 ? C - 2 : 0);
  for (int l = C - 1; l >= 1; --l) {
    cx<R> nn = shfl_el(gk, l >= 2 ? l - 2 : 0);
    const cx<R> h = cscale(cur, lane_value(isql, l));
    h0 = csel(lane == l, h, h0);
    cfma_conj(nxt, b1, h);
    cfma_conj(nn, a11, cscale(h, lane_value(sql, l - 1)));   // weight 0 at l = 1
    cur = nxt;
    nxt = nn;
  }
  add(3, h0, shfl_el(f0, lane > 0 ? lane - 1 : 0));
  const R wl = lane_value(sql, max(lane - 1, 0));   // 0 at l = 1
  add(4, h0, cscale(shfl_el(f0, max(lane - 2, 0)), wl));
  // butterfly sums over the wavefront (fixed order), lane 0 adds to the slot
  const int at[5] = {npos, 0, 1, NR + npos, NR + 1};
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    double vx = sx[i], vy = sy[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      vx += __shfl_xor(vx, off, 64);
      vy += __shfl_xor(vy, off, 64);
    }
    if (lane == 0) {
      const double2 v = slot[at[i]];
      slot[at[i]] = make_double2(v.x + vx, v.y + vy);
    }
  }
  if (lane == 0) st(cbar, cur);
}

// Final: sum the partial slots in order, symmetrise Abar, scatter to the
// caller's block order (zero for dropped modes), write dc.
struct FinalArgs {
  int blk2pos[2 * kMaxModes];
  int M2, npos;
};

template <typename R>
__global__ __launch_bounds__(kThreads) void k_vjp_final(const double2* __restrict__ partial, int nslots, FinalArgs a,
                                                        const cx<R>* __restrict__ cbar, cx<R>* dA, cx<R>* db,
                                                        cx<R>* dc) {
  __shared__ double2 red[kThreads];
  const int NR = a.npos + 1, P = a.npos * NR;
  const int idx = blockIdx.x;
  int c1 = -1, c2 = -1;   // pair columns summed (c2: transpose for the symmetric part)
  if (idx < a.M2 * a.M2) {
    const int p = a.blk2pos[idx / a.M2], q = a.blk2pos[idx % a.M2];
    if (p >= 0 && q >= 0) {
      c1 = p * NR + q;
      c2 = q * NR + p;
    }
  } else if (idx < a.M2 * a.M2 + a.M2) {
    const int p = a.blk2pos[idx - a.M2 * a.M2];
    if (p >= 0) c1 = p * NR + a.npos;
  }
  double sx = 0.0, sy = 0.0;
  // slots threadIdx.x, + kThreads, ... in order, KS of them per pass: their
  // loads go out before the first add
  constexpr int KS = 8;
  if (c1 >= 0) {
    for (int s0 = threadIdx.x; s0 < nslots; s0 += KS * kThreads) {
      double2 v[KS], w[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const size_t s = s0 + k * kThreads;
        const bool in = (int)s < nslots;
        v[k] = in ? partial[s * P + c1] : make_double2(0.0, 0.0);
        w[k] = in && c2 >= 0 ? partial[s * P + c2] : make_double2(0.0, 0.0);
      }
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        sx += v[k].x + w[k].x;
        sy += v[k].y + w[k].y;
      }
    }
  }
  red[threadIdx.x] = make_double2(sx, sy);
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      red[threadIdx.x].x += red[threadIdx.x + w].x;
      red[threadIdx.x].y += red[threadIdx.x + w].y;
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  const double2 t = red[0];
  if (idx < a.M2 * a.M2)
    st(dA + idx, cmake<R>((R)(0.5 * t.x), (R)(0.5 * t.y)));
  else if (idx < a.M2 * a.M2 + a.M2)
    st(db + (idx - a.M2 * a.M2), cmake<R>((R)t.x, (R)t.y));
  else
    st(dc, ld(cbar));
}

// ---------------------------------------------------------------------------
// Block levels: the translation unit for the plan's detected modes.
// ---------------------------------------------------------------------------
template <typename R, int LO>
hipError_t launch_vjp_block_range(const Plan& Pl, const DevPlan& P, const VjpPtrs<R>& Vp, const cx<R>* Ai,
                                  const cx<R>* bi, int S, int nwork, double2* partial, hipStream_t st);
template <typename R>
hipError_t launch_vjp_block_level(const Plan& Pl, const DevPlan& P, const VjpPtrs<R>& Vp, const cx<R>* Ai,
                                  const cx<R>* bi, int S, int nwork, double2* partial, hipStream_t st) {
  return Pl.MD <= 4 ? launch_vjp_block_range<R, 1>(Pl, P, Vp, Ai, bi, S, nwork, partial, st)
                    : launch_vjp_block_range<R, 5>(Pl, P, Vp, Ai, bi, S, nwork, partial, st);
}

// Workgroups of a block level (streamed rows: private slots for at most kStreamSlots workgroups)
int vjp_block_grid(const Plan& Pl, int nwork) {
  return (int)std::min<int64_t>((int64_t)nwork * vjp_geo(Pl, nwork).nchunks,
                                Pl.st_vjp ? kStreamSlots : kPartialSlots - 1);
}

// ---------------------------------------------------------------------------
// host orchestration
// ---------------------------------------------------------------------------
template <typename R>
static const cx<R>* fptr(const Plan& Pl, const char* base, size_t off, int g, int S) {
  if (S < 0 || off == 0) return nullptr;
  return reinterpret_cast<const cx<R>*>(base + off +
                                         (size_t)Pl.lvl[(size_t)g * (Pl.smax + 2) + S] * Pl.B * sizeof(cx<R>));
}
template <typename R>
static cx<R>* gptr(const Plan& Pl, char* base, size_t off, int g, int S) {
  if (S < 0 || off == 0) return nullptr;
  return reinterpret_cast<cx<R>*>(base + off + (size_t)(S & 1) * Pl.maxN[g] * Pl.B * sizeof(cx<R>));
}

template <typename R>
static hipError_t run_vjp_t(const Plan& Pl, bool odd, const void* A, const void* b, const void* c,
                            const void* saved, const void* drho, void* dA, void* db, void* dc, char* ws,
                            hipStream_t st) {
  const VjpLayout V = vjp_layout(Pl, odd, 0);
  const FwdLayout Ls = fwd_layout(Pl, true, true, 0);
  const char* sv = reinterpret_cast<const char*>(saved);
  cx<R>* Ai = reinterpret_cast<cx<R>*>(ws + V.prep);
  cx<R>* bi = Ai + (size_t)Pl.npos * Pl.npos;
  cx<R>* cb = bi + Pl.npos;   // reused: holds cbar at the end
  double2* partial = reinterpret_cast<double2*>(ws + V.partial);
  hipError_t e = hipSuccess;
  const int MD = Pl.MD;
  // Checkpointed plans: the forward values of one segment of levels at a
  // time, recomputed from the segment's checkpoint into the segment buffer
  // (slot k holds level seg_lo - 1 + k); F0 of every level is in `saved`.
  const bool ck = Pl.ckpt > 0;
  const CkptLayout Lc = ck ? ckpt_layout(Pl) : CkptLayout();
  const SegLayout Sg = ck ? seg_layout(Pl) : SegLayout();
  const size_t f0off = ck ? Lc.f0 : Ls.f0;
  auto used = [&](int f) { return ckpt_keeps_family(Pl, f) && (odd || f >= 1 + 2 * MD); };
  // level L of family f in the segment buffer (levels seg_lo - 1 .. held)
  auto seg_slot = [&](int f, int lo, int L) {
    return reinterpret_cast<cx<R>*>(ws + Sg.fam[f] +
                                    (size_t)seg_node(Pl, Pl.fam_group[f], lo, L) * Pl.B * sizeof(cx<R>));
  };
  // the checkpoint below segment lo > 0
  auto ck_level = [&](int f, int lo) {
    return reinterpret_cast<const cx<R>*>(sv + Lc.ck[(size_t)(lo / Pl.ckpt - 1) * Pl.nfam + f]);
  };
  // forward values of levels lo..hi from the checkpoint below lo (`whole`: which
  // then stands before them in the segment buffer)
  auto restore = [&](int lo, int hi, bool whole) -> hipError_t {
    if (lo > 0 && whole) {
      const void* src[kMaxFam] = {};
      void* dst[kMaxFam] = {};
      int64_t n[kMaxFam] = {};
      for (int f = 1; f < Pl.nfam; ++f) {
        if (!used(f)) continue;
        src[f] = ck_level(f, lo);
        dst[f] = seg_slot(f, lo, lo - 1);
        n[f] = Pl.ncnt[(size_t)Pl.fam_group[f] * (Pl.smax + 1) + lo - 1] * Pl.B;
      }
      const hipError_t x = launch_copy_fams(Pl, src, dst, n, st);
      if (x != hipSuccess) return x;
    }
    const cx<R>* f0all = reinterpret_cast<const cx<R>*>(sv + f0off);
    for (int L = lo; L <= hi; ++L) {
      const void* rd[kMaxFam] = {};
      void* wr[kMaxFam] = {};
      for (int f = 1; f < Pl.nfam; ++f) {
        if (!used(f)) continue;
        rd[f] = L > lo ? seg_slot(f, lo, L - 1) : L > 0 ? ck_level(f, lo) : nullptr;
        wr[f] = seg_slot(f, lo, L);
      }
      // F0 of level L + 1 is written again with the values it already holds
      cx<R>* f0nxt = L < Pl.smax ? const_cast<cx<R>*>(f0all) + (size_t)Pl.lvl[L + 1] * Pl.B : nullptr;
      KTimer kt(Pl, KK_FWD_LEVEL, st);
      const hipError_t x = launch_fwd_level(Pl, odd, L, rd, wr, f0all + (size_t)Pl.lvl[L] * Pl.B, f0nxt, Ai, bi, st);
      if (x != hipSuccess) return x;
    }
    return hipSuccess;
  };
  if (!Pl.small_vjp || ck) {
    KTimer kt(Pl, KK_PREP, st);
    e = launch_prep(Pl, A, b, c, Ai, nullptr, st);
  }
  if (e != hipSuccess) return e;
  if (Pl.small_vjp) {
    void *fam[kMaxFam] = {}, *gfam[kMaxFam] = {};
    for (int f = 0; f < Pl.nfam; ++f) gfam[f] = V.gfam[f] ? ws + V.gfam[f] : nullptr;
    fam[0] = const_cast<char*>(sv) + f0off;
    const int every = ck ? Pl.ckpt : Pl.smax + 1;
    for (int lo = Pl.smax / every * every; lo >= 0; lo -= every) {
      const int hi = std::min(lo + every - 1, Pl.smax);
      if (ck && (e = restore(lo, hi, true)) != hipSuccess) return e;
      for (int f = 1; f < Pl.nfam; ++f) {
        // a segment buffer starts with level lo - 1: its node 0 is that many
        // nodes before it
        const int64_t skip = ck ? Pl.lvl[(size_t)Pl.fam_group[f] * (Pl.smax + 2) + std::max(lo - 1, 0)] : 0;
        const bool have = ck ? used(f) : Ls.fam[f] != 0;
        fam[f] = !have ? nullptr
                 : ck  ? reinterpret_cast<cx<R>*>(ws + Sg.fam[f]) - skip
                       : reinterpret_cast<cx<R>*>(const_cast<char*>(sv) + Ls.fam[f]);
      }
      KTimer kt(Pl, KK_VJP_LEVEL, st);
      if ((e = launch_point_small_vjp<R>(Pl, make_devplan(Pl, odd), odd, static_cast<const cx<R>*>(A),
                                         static_cast<const cx<R>*>(b), static_cast<const cx<R>*>(c), Ai, fam, gfam,
                                         static_cast<const cx<R>*>(drho), reinterpret_cast<cx<R>*>(ws + V.g0),
                                         static_cast<cx<R>*>(dA), static_cast<cx<R>*>(db), static_cast<cx<R>*>(dc), hi,
                                         lo, reinterpret_cast<double*>(partial), st)) != hipSuccess)
        return e;
    }
    return hipSuccess;
  }
  const int PP = Pl.npos * (Pl.npos + 1);
  // reduction slots in use: one per workgroup of the largest level, and the
  // undetected-block fill's (the last one)
  int nslots = Pl.B > 1 ? 1 : 0;
  for (int S = 0; S <= Pl.smax && Pl.MD > 0; ++S)
    nslots = std::max(nslots, (Pl.B > 1 ? 1 + vjp_block_grid(Pl, (int)Pl.ncnt[S]) : vjp_point_grid(Pl, S)));
  const int64_t npart = (int64_t)nslots * PP;
  {
    KTimer kt(Pl, KK_ZERO, st);
    hipLaunchKernelGGL(k_zero_d2, dim3((unsigned)std::min<int64_t>(std::max<int64_t>(1, (npart + 255) / 256), 4096)), dim3(256), 0, st,
                       partial, npart);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  DevPlan P = make_devplan(Pl, odd);
  cx<R>* g0 = reinterpret_cast<cx<R>*>(ws + V.g0);
  if (Pl.level_cap >= 0) {
    // a total photon cutoff: the cotangent already comes in level (node) order
    KTimer kt(Pl, KK_PERM_IN, st);
    if ((e = hipMemcpyAsync(g0, drho, (size_t)Pl.nodes_total * sizeof(cx<R>), hipMemcpyDeviceToDevice, st)) !=
        hipSuccess)
      return e;
  } else {
    const int64_t total = Pl.out_elems;
    const int64_t tiles = ((Pl.nodes_total + kOutTN - 1) / kOutTN) * ((Pl.B + kOutTK - 1) / kOutTK);
    const int ept = total >= kOutEPTMin ? kOutEPT : 1;
    const int64_t grid = std::min<int64_t>(Pl.B > 1 ? tiles : (total + kThreads * ept - 1) / (kThreads * ept), 65536);
    const size_t shm = 16 * ((((size_t)(Pl.MD + 1) * (Pl.smax + 3)) * 4 + 15) / 16) +
                       16 * (((size_t)(Pl.smax + 2) * 8 + 15) / 16) +
                       (Pl.B > 1 ? (size_t)kOutTN * (kOutTK + 1) * sizeof(cx<R>) : 0);
    KTimer kt(Pl, KK_PERM_IN, st);
    auto* kfn = ept == 1 ? &k_perm_in<R, 1> : &k_perm_in<R, kOutEPT>;
    hipLaunchKernelGGL(kfn, dim3(grid), dim3(kThreads), shm, st, P,
                       reinterpret_cast<const cx<R>*>(drho), g0, (int64_t)Pl.nodes_total, total);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (Pl.level_cap >= 0 && MD > 0) {
    // under a total photon cutoff the families of the last level feed no
    // target: their cotangents (read by that level's pivots) start at zero
    for (int f = 1; f < Pl.nfam; ++f) {
      if (V.gfam[f] == 0) continue;
      const int g = Pl.fam_group[f];
      const int64_t n = Pl.maxN[g] * Pl.B;
      hipLaunchKernelGGL((k_zero_cx<R>), dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, st,
                         gptr<R>(Pl, ws, V.gfam[f], g, Pl.smax), n);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  int seg_lo = Pl.smax + 1;
  for (int S = Pl.smax; S >= 0 && MD > 0; --S) {
    if (ck && S < seg_lo) {
      seg_lo = (S / Pl.ckpt) * Pl.ckpt;
      if ((e = restore(seg_lo, S, false)) != hipSuccess) return e;
    }
    VjpPtrs<R> Vp;
    std::memset(&Vp, 0, sizeof(Vp));
    for (int f = 0; f < Pl.nfam; ++f) {
      const int g = Pl.fam_group[f];
      if (!ck || f == 0) {
        const size_t foff = f == 0 ? f0off : Ls.fam[f];
        Vp.fprev[f] = fptr<R>(Pl, sv, foff, g, S - 1);
        Vp.fcur[f] = fptr<R>(Pl, sv, foff, g, S);
      } else if (used(f)) {
        Vp.fprev[f] = S > seg_lo ? seg_slot(f, seg_lo, S - 1) : S > 0 ? ck_level(f, seg_lo) : nullptr;
        Vp.fcur[f] = seg_slot(f, seg_lo, S);
      }
      Vp.gprev[f] = gptr<R>(Pl, ws, V.gfam[f], g, S - 1);
      Vp.gcur[f] = gptr<R>(Pl, ws, V.gfam[f], g, S);
    }
    Vp.gf0nxt = (Pl.level_cap >= 0 && S == Pl.smax) ? nullptr : gptr<R>(Pl, ws, V.gfam[0], 0, S + 1);
    // every level kernel reads these unconditionally
    if (!Vp.fcur[0] || !Vp.gcur[0]) return hipErrorInvalidValue;
    Vp.d0cur = reinterpret_cast<const cx<R>*>(reinterpret_cast<const char*>(g0) +
                                              (size_t)Pl.lvl[S] * Pl.B * sizeof(cx<R>));
    Vp.node = Pl.d_node ? Pl.d_node + (size_t)Pl.lvl[S] * kNodeStride : nullptr;
    Vp.priv = V.priv ? reinterpret_cast<cx<R>*>(ws + V.priv) : nullptr;
    Vp.priv_stride = (int64_t)vjp_private_entries(Pl);
    const int nwork = (int)Pl.ncnt[S];
    KTimer kt(Pl, KK_VJP_LEVEL, st);
    if (Pl.B == 1) {
      if ((e = launch_vjp_point_level<R>(Pl, P, odd, S, Vp, Ai, bi, nwork, partial, st)) != hipSuccess) return e;
    } else {
      if ((e = launch_vjp_block_level<R>(Pl, P, Vp, Ai, bi, S, nwork, partial, st)) != hipSuccess) return e;
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // cotangent of the seed block: F0 ring slot of level 0 (MD > 0) or drho itself
  const cx<R>* gseed = MD > 0 ? gptr<R>(Pl, ws, V.gfam[0], 0, 0) : g0;
  const cx<R>* cbar_src = gseed;
  if (Pl.B > 1) {
    const cx<R>* G0blk = reinterpret_cast<const cx<R>*>(sv + f0off);
    KTimer kt(Pl, KK_UFILL_VJP, st);
    const size_t shm = ufill_launch_lds_bytes(Pl, true);
    if (shm > kMaxLds) return hipErrorInvalidConfiguration;
    // streamed: the block's cotangents accumulate in the workspace
    cx<R>* gbuf = Pl.st_ufill_vjp ? reinterpret_cast<cx<R>*>(ws + V.ublk) : nullptr;
    if (Pl.st_ufill_vjp && V.ublk == 0) return hipErrorInvalidValue;
    double2* slot = partial + (size_t)(nslots - 1) * PP;
    if (Pl.nq == 2) {
      hipLaunchKernelGGL((k_ufill_vjp_rows<R>), dim3(1), dim3(64), 0, st, P, Ai, bi, G0blk, gseed, slot, cb);
    } else {
      auto* kfn = Pl.st_ufill_vjp ? (Pl.nq == 4 ? &k_ufill_vjp<R, 4, true> : &k_ufill_vjp<R, 6, true>)
                                  : (Pl.nq == 4 ? &k_ufill_vjp<R, 4, false> : &k_ufill_vjp<R, 6, false>);
      if (shm > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)shm);
      hipLaunchKernelGGL(kfn, dim3(1), dim3(64), shm, st, P, Ai, bi, G0blk, gseed, Pl.d_elist, Pl.d_woff, Pl.wmax,
                         slot, cb, gbuf);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    cbar_src = cb;
  }
  FinalArgs fa;
  std::memset(&fa, 0, sizeof(fa));
  for (int u = 0; u < 2 * Pl.M; ++u) fa.blk2pos[u] = -1;
  for (int p = 0; p < Pl.npos; ++p) fa.blk2pos[Pl.pos2blk[p]] = p;
  fa.M2 = 2 * Pl.M;
  fa.npos = Pl.npos;
  const int nout = fa.M2 * fa.M2 + fa.M2 + 1;
  KTimer kt(Pl, KK_VJP_FINAL, st);
  hipLaunchKernelGGL((k_vjp_final<R>), dim3(nout), dim3(kThreads), 0, st, partial, nslots, fa, cbar_src,
                     reinterpret_cast<cx<R>*>(dA), reinterpret_cast<cx<R>*>(db), reinterpret_cast<cx<R>*>(dc));
  return hipGetLastError();
}

hipError_t run_vjp(const Plan& Pl, bool odd, const void* A, const void* b, const void* c, const void* saved,
                   const void* drho, void* dA, void* db, void* dc, void* ws, hipStream_t st) {
  if (Pl.dt == FD_C64) return run_vjp_t<float>(Pl, odd, A, b, c, saved, drho, dA, db, dc, (char*)ws, st);
  return run_vjp_t<double>(Pl, odd, A, b, c, saved, drho, dA, db, dc, (char*)ws, st);
}

}  // namespace fd
