// Point units (every mode detected, Algorithm 1) on the matrix cores.
//
// A pivot application at a lattice point is y = A x: x the 2 MD reads of the
// pivot (scaled by sqrt(p_l)), y its targets (scaled by 1 / sqrt(p_i + 1)).  A is
// the same at every point, so the points of a level are the columns of a
// [NP x NP] [NP x points] product.  A wavefront takes 16 points at a time:
// lane (c, kq) = (lane & 15, lane >> 4) holds the reads at positions p = 4 s + kq,
// s = 0..ceil(NP / 4) - 1, of point c -- the B operand of the 16x16x4 MFMA -- and
// gets the targets at the same positions of the same point (the gfx950 output
// layout; the rows of A are permuted in single precision, whose output rows
// lie the other way round), so A sits in 4 ceil(NP / 4) registers per lane
// and neither operand goes through the LDS.  One point per lane kept 2 x 16
// complex registers of reads and targets live and fetched A through scalar
// loads, ceil(NP^2 / 4) cache lines per wavefront and pivot with a wait each.
//
// Ranks: the ranks of the neighbours and the digits of m go through LDS rows,
// from which the four lanes of a point take the modes of their positions; one
// point per lane and 64-point tile (T = 4, large levels of the reverse sweep) or
// the four lanes of a 16-point tile's point alike (T = 1).
#pragma once

#include "fwd_units.h"

namespace fd {

template <typename R>
struct Mma;
template <>
struct Mma<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // position held by row r of the A operand, so that output register s of
  // lane (c, kq) is position 4 s + kq
  static __device__ __forceinline__ int row_pos(int r) { return r; }
};
template <>
struct Mma<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row_pos(int r) { return 4 * (r & 3) + (r >> 2); }
};

template <typename T>
__device__ __forceinline__ T* global_at(uint64_t a) {
  return (T*)(__attribute__((address_space(1))) T*)a;
}

constexpr int kPtPos = 16;                 // positions of one MFMA tile (2 MD <= 16)
// pointer table rows: bridge K = 0..MD-1, then the diagonal pivot
constexpr int pt_table_entries(int MD) { return (MD + 1) * kPtPos; }
// ints of one wavefront's rank rows: rank(m - 1_j), rank(m + 1_j), digits of m
constexpr int pt_row_ints(int MD, int T) { return (2 * MD + 2) * 16 * T; }

// Square-root tables and PN table of the plan, from its device copy.
template <typename R>
__device__ __forceinline__ void pt_load_tables(const DevPlan& P, int MD, R* sq, int* spn) {
  const R* t = reinterpret_cast<const R*>(P.sqt);
  const int* pn = P.pn;
  for (int i = threadIdx.x; i < 2 * (kMaxCut + 4); i += blockDim.x) sq[i] = t[i];
  const int n = (MD + 1) * P.pnw;
  for (int i = threadIdx.x; i < n; i += blockDim.x) spn[i] = pn[i];
}

// Digits (8 bits each, mode j at bit 8 j) and neighbour ranks of lattice
// point r of level S into slot q of the wavefront's rows.
template <int MD, int T>
__device__ __forceinline__ void pt_rank_rows(const DevPlan& P, const int* spn, const uint64_t* mt, int S, int r, int q,
                                             int* rows) {
  constexpr int SL = 16 * T;
  int m[MD], s[MD + 1], rdn[MD], rup[MD];
  uint64_t pk = 0;
  if (mt) {
    pk = mt[r];
    s[0] = S;
#pragma unroll
    for (int d = 0; d < MD; ++d) {
      m[d] = (int)((pk >> (8 * d)) & 255);
      s[d + 1] = s[d] - m[d];
    }
  } else {
    unrank<MD>(spn, P.pnw, P.CD, S, r, m, s);
#pragma unroll
    for (int d = 0; d < MD; ++d) pk |= (uint64_t)m[d] << (8 * d);
  }
  neighbour_ranks<MD>(spn, P.pnw, s, rdn, rup);
#pragma unroll
  for (int j = 0; j < MD; ++j) {
    rows[j * SL + q] = rdn[j];
    rows[(MD + j) * SL + q] = rup[j];
  }
  reinterpret_cast<uint64_t*>(rows + 2 * MD * SL)[q] = pk;
}
template <int MD, int T>
__device__ __forceinline__ uint64_t pt_digits(const int* rows, int q) {
  return reinterpret_cast<const uint64_t*>(rows + 2 * MD * 16 * T)[q];
}

// A as the A operand (conj^T = 1: its conjugate transpose): entry [row][4 s + kq].
template <int MD, typename R>
struct PtMat {
  static constexpr int NP = 2 * MD, KS = (NP + 3) / 4;
  R ar[KS], ai[KS];
  __device__ __forceinline__ void load(const cx<R>* __restrict__ A, bool adjoint) {
    const int lane = threadIdx.x & 63;
    const int row = Mma<R>::row_pos(lane & 15), kq = lane >> 4;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int col = 4 * s + kq;
      const bool in = row < NP && col < NP;
      const cx<R> v = ld(A + (in ? (adjoint ? col * NP + row : row * NP + col) : 0));
      ar[s] = in ? v.x : R(0);
      ai[s] = in ? (adjoint ? -v.y : v.y) : R(0);
    }
  }
  // (re, im) += M x over the positions
  __device__ __forceinline__ void apply(const cx<R> (&x)[KS], typename Mma<R>::v4& re, typename Mma<R>::v4& im) const {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      re = Mma<R>::mma(ar[s], x[s].x, re);
      im = Mma<R>::mma(ar[s], x[s].y, im);
      re = Mma<R>::mma(ai[s], -x[s].y, re);
      im = Mma<R>::mma(ai[s], x[s].x, im);
    }
  }
};

// LDS tables of a workgroup for one level.
template <typename R>
struct PtLds {
  const R* sq;
  const R* isq;
  const int* spn;
  const uint64_t* rd;      // read pointers [(MD + 1) x 16]
  const uint64_t* wr;      // write pointers
};

// Pointer tables of the forward step from L.rd / L.wr (see LevelPtrs): what
// position p of pivot row K reads and writes.
template <int MD, bool ODD, typename R, typename LP>
__device__ __forceinline__ void pt_fill_pointers(const LP& L, uint64_t* rd, uint64_t* wr) {
  constexpr int NP = 2 * MD;
  for (int t = threadIdx.x; t < pt_table_entries(MD); t += blockDim.x) {
    const int K = t / kPtPos, p = t % kPtPos, j = p >> 1, b = p & 1;
    int fr = 0, fw = 0;   // 0: F0 (current level read, next level written)
    if (p < NP) {
      if (K == MD) {
        if (!ODD) continue;
        fr = b ? fam_f1k(j) : fam_f1b(MD, j);
        fw = b ? fam_f1b(MD, j) : fam_f1k(j);
      } else if (p == 2 * K) {
        fw = fam_f2(MD, K);
      } else if (p == 2 * K + 1) {
        fr = fam_f2(MD, K);
      } else if (j > K) {
        fr = b ? fam_1010(MD, K, j) : fam_1001(MD, K, j);
        fw = b ? fam_1001(MD, K, j) : fam_1010(MD, K, j);
      }
    }
    const cx<R>* a = fr ? L.rd[fr] : L.f0cur;
    cx<R>* w = fw ? L.wr[fw] : L.f0nxt;
    rd[t] = reinterpret_cast<uint64_t>(a);
    wr[t] = reinterpret_cast<uint64_t>(w);
  }
}

// A lane's constants: A in operand layout, b and the cutoffs of the modes at its
// positions; with tangents (DUAL, forward mode) dA and db too.
template <int MD, bool ODD, bool DUAL, typename R>
struct PtConst {
  static constexpr int KS = PtMat<MD, R>::KS;
  PtMat<MD, R> A, dA;
  cx<R> b[KS], db[KS];
  int cj[KS];
  // dT: bytes from a value to its tangent
  __device__ __forceinline__ void load(const DevPlan& P, const cx<R>* __restrict__ Ai, const cx<R>* __restrict__ bi,
                                       int64_t dT) {
    const int kq = (threadIdx.x & 63) >> 4;
    A.load(Ai, false);
    if (DUAL) dA.load(tangent_of(Ai, dT), false);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      cj[s] = P.CD[min(2 * s + (kq >> 1), MD - 1)];
      const bool in = ODD && 4 * s + kq < 2 * MD;
      b[s] = in ? ld(bi + 4 * s + kq) : czero<R>();
      if (DUAL) db[s] = in ? ld(tangent_of(bi, dT) + 4 * s + kq) : czero<R>();
    }
  }
};

// The work of a forward level: items (K, tile of 16 points) for every bridge K,
// whose points are the first n[K] of the level (n_<K = 0).  One item applies
// bridge K; the K = 0 items also apply the diagonal pivot, the others only
// form its value at position 2 K (ODD).  A tile whose points take every bridge
// would otherwise run them one after the other: on the first level of eight
// modes 14 us against 6.
struct PtItems {
  int n[kMaxD];
  __host__ __device__ __forceinline__ int tiles(int K) const { return (n[K] + 15) >> 4; }
};
// Item u: its bridge, first point and the bridge's number of points.
template <int MD>
__device__ __forceinline__ bool pt_item(const PtItems& I, int u, int* K, int* base, int* n) {
  bool found = false;
#pragma unroll
  for (int k = 0; k < MD; ++k) {
    const int t = I.tiles(k);
    if (!found && u < t) {
      found = true;
      *K = k;
      *base = 16 * u;
      *n = I.n[k];
    }
    u -= t;
  }
  return found;
}

// One item: 16 lattice points base.. of level S (the n points of bridge K), one
// wavefront.  DUAL carries every amplitude's tangent along (Sec. 2.5, the
// tangent recurrences summed along one direction): with x, y the values and
// x', y' their tangents,
//   y' ~ A x' + dA x + b p' + db p
// for the same reads, targets and scales (p the pivot's value).
template <int MD, bool ODD, bool DUAL, typename R>
__device__ __forceinline__ void fwd_point_item(const DevPlan& P, const PtLds<R>& Y, const PtConst<MD, ODD, DUAL, R>& C,
                                               const cx<R>* f0cur, bool has_next, const uint64_t* mt, int S, int K,
                                               int base, int n, int* rows, int64_t dT = 0) {
  constexpr int NP = 2 * MD, KS = PtMat<MD, R>::KS;
  typedef typename Mma<R>::v4 v4;
  const int lane = threadIdx.x & 63, c = lane & 15, kq = lane >> 4, hk = kq >> 1, side = kq & 1;
  const bool live = base + c < n;
  const int r = min(base + c, n - 1);
  pt_rank_rows<MD, 1>(P, Y.spn, mt, S, r, c, rows);
  wave_sync();
  {
    const uint64_t pk = pt_digits<MD, 1>(rows, c);
    int mj[KS], dn[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int j = 2 * s + hk;
      mj[s] = (int)((pk >> (8 * j)) & 255);
      dn[s] = rows[min(j, MD - 1) * 16 + c];
    }
    const cx<R> g0 = ld(f0cur + r);
    cx<R> t0 = czero<R>();
    if (DUAL) t0 = ld(tangent_of(f0cur, dT) + r);
    // the reads of pivot row K at this lane's positions; absent ones read the
    // level's first F0 entry and are discarded, so every load is issued
    // unconditionally and a pivot's loads share one wait
    auto reads = [&](int K, bool valid, cx<R>(&x)[KS], cx<R>(&tx)[KS]) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int p = 4 * s + kq;
        const bool first = p == 2 * K;   // never for the diagonal row (2 MD > p)
        const bool ok = valid && p < NP && (first || ((p > 2 * K || K == MD) && mj[s] > 0));
        const cx<R>* a = global_at<const cx<R>>(Y.rd[K * kPtPos + p]) + (first ? r : dn[s]);
        a = ok ? a : f0cur;
        const R w = Y.sq[mj[s] + (first ? 1 : 0)];
        const cx<R> v = ld(a);
        if (DUAL) {
          const cx<R> u = ld(tangent_of(a, dT));
          tx[s] = cscale(csel(ok, u, czero<R>()), w);
        }
        x[s] = cscale(csel(ok, v, czero<R>()), w);
      }
    };
    // targets of a pivot of value p (tangent tp) with reads x (tx)
    auto product = [&](const cx<R>& p, const cx<R>& tp, const cx<R>(&x)[KS], const cx<R>(&tx)[KS], v4& re, v4& im,
                       v4& tre, v4& tim) {
#pragma unroll
      for (int s = 0; s < 4; ++s) re[s] = im[s] = tre[s] = tim[s] = R(0);
      if (ODD) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          cx<R> v = czero<R>();
          cfma(v, C.b[s], p);
          re[s] = v.x;
          im[s] = v.y;
          if (DUAL) {
            cx<R> u = czero<R>();
            cfma(u, C.db[s], p);
            cfma(u, C.b[s], tp);
            tre[s] = u.x;
            tim[s] = u.y;
          }
        }
      }
      C.A.apply(x, re, im);
      if (DUAL) {
        C.dA.apply(x, tre, tim);
        C.A.apply(tx, tre, tim);
      }
    };
    auto write = [&](int K, int s, int idx, const cx<R>& v, const cx<R>& tv) {
      cx<R>* dst = global_at<cx<R>>(Y.wr[K * kPtPos + 4 * s + kq]) + idx;
      st(dst, v);
      if (DUAL) st(tangent_of(dst, dT), tv);
      count_write(P, dst);
    };
    cx<R> y[KS], ty[KS];
    if (ODD) {
      // diagonal pivot d(m): reads d(m) - 1_l, writes d(m) + 1_i
      const bool valid = live && (int)(pk & 255) <= P.CD[0] - 2;
      cx<R> x[KS], tx[KS];
      reads(MD, valid, x, tx);
      v4 re, im, tre, tim;
      product(g0, t0, x, tx, re, im, tre, tim);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int p = 4 * s + kq, j = 2 * s + hk;
        const R w = Y.isq[mj[s] + 1];
        y[s] = cscale(cmake<R>(re[s], im[s]), w);
        if (DUAL) ty[s] = cscale(cmake<R>(tre[s], tim[s]), w);
        const int room = (j == 0 ? C.cj[s] - 2 - side : C.cj[s] - 2) - mj[s];
        if (K == 0 && valid && p < NP && room >= 0) write(MD, s, r, y[s], ty[s]);
      }
    }
    const int mK = (int)((pk >> (8 * K)) & 255);
    const bool valid = live && mK <= P.CD[K] - 2;
    if (__ballot(valid) != 0ull) {
      // pivot d(m) + 1_ket(K)
      cx<R> x[KS], tx[KS];
      reads(K, valid, x, tx);
      const int up = rows[(MD + K) * 16 + c];
      cx<R> yk = czero<R>(), tyk = czero<R>();
      if (ODD) {
        // the pivot value: target 2 K of the diagonal pivot, held by lane
        // (c, 2 (K & 1)) in register K / 2
        const int src = c + 32 * (K & 1);
        yk = y[0];
        if (DUAL) tyk = ty[0];
#pragma unroll
        for (int s = 1; s < KS; ++s)
          if ((K >> 1) == s) {
            yk = y[s];
            if (DUAL) tyk = ty[s];
          }
        yk = cmake<R>(__shfl(yk.x, src), __shfl(yk.y, src));
        if (DUAL) tyk = cmake<R>(__shfl(tyk.x, src), __shfl(tyk.y, src));
      }
      v4 re, im, tre, tim;
      product(yk, tyk, x, tx, re, im, tre, tim);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int p = 4 * s + kq;
        const int two = p == 2 * K ? 1 : 0;
        const bool nxt = p == 2 * K + 1;   // d(m + 1_K): none above the last level (a total photon cutoff)
        const bool ok = valid && p < NP && p >= 2 * K && mj[s] + two <= C.cj[s] - 2 && (!nxt || has_next);
        const R w = Y.isq[mj[s] + 1 + two];
        if (ok)
          write(K, s, nxt ? up : r, cscale(cmake<R>(re[s], im[s]), w),
                DUAL ? cscale(cmake<R>(tre[s], tim[s]), w) : czero<R>());
      }
    }
  }
  wave_sync();   // the rows are rewritten by the next item
}

// The items of level S (group K's points of a level are those with n_<K = 0).
inline PtItems pt_items(const Plan& Pl, int S) {
  PtItems I = {};
  for (int K = 0; K < Pl.MD; ++K) I.n[K] = (int)Pl.ncnt[(size_t)K * (Pl.smax + 1) + S];
  return I;
}

// LDS bytes of the point kernels' tables and rank rows (`waves` wavefronts).
inline size_t pt_lds_bytes(const Plan& Pl, int T, int waves, int tables) {
  const size_t rb = elem_bytes(Pl.dt) / 2;
  const size_t pn = ((size_t)(Pl.MD + 1) * (Pl.smax + 3) * 4 + 15) / 16 * 16;
  return 2 * (kMaxCut + 4) * rb + pn + (size_t)tables * pt_table_entries(Pl.MD) * 8 +
         (size_t)waves * pt_row_ints(Pl.MD, T) * 4;
}

}  // namespace fd
