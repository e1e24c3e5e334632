// Reverse step of plans with every mode detected (Algorithm 1): the points of a
// level in tiles of 16 columns on the matrix cores.
//
// Per pivot, with h the (scaled) cotangents of its targets and x its reads:
//   u = A^H h            the cotangents of the reads, written to their only reader's slot
//   D += h conj(x)^T     Abar, summed over every point
// Both are contractions.  The first has A^H as the stationary operand in
// registers, like the forward (pt_units.h): lane (c, kq) loads the cotangents at
// positions 4 s + kq of point c and gets u at the same positions.  The second
// contracts over the points, so its operands need position lane & 15 of points
// 4 s + kq: the reads x are loaded from memory in that layout (64-byte runs of
// four points; nothing else uses them), h is turned through a 16 x 17 LDS tile.  Its
// complex product takes three real ones (see vjp_common.h).  Up to seven modes the
// pivot's value joins x as position 2 MD and conj(b) joins A^H as row 2 MD, so bbar
// and b^H h come out of the same products; eight modes fill the tile and form
// both on the vector unit.
//
// What bounds it: 48 bytes per computed amplitude, which the counters put at 1.25x;
// the large levels of eight modes of cutoff 8 move 495 MB in 134 us, 3.7 TB/s (a
// large copy on this card: 4.9).  Loading a tile's first bridge before the products
// of the tile before it made no difference (3608 against 3620 us).  With one point
// per lane the two 16-vectors and the reduction's staging held 202 VGPRs + 17 KB of
// LDS per wavefront (two wavefronts per SIMD, 60 % of their cycles waiting): 5.24 ms
// per reverse sweep, now 4.06.
#pragma once

#include "vjp_common.h"

namespace fd {

// A level of the reverse sweep in LDS and pointers: pointer tables of
// pt_fill_vjp_pointers (xp: then the values of the pivots F1k(K)), tables, F0 of
// the level, its cotangents from the output (d0) and where their sums go (g0).
template <typename R>
struct VjpPtLevel {
  const uint64_t *hp, *gp, *xp;
  const R *sq, *isq;
  const int* spn;
  const cx<R>*f0, *d0;
  cx<R>* g0;
  bool has_next;   // false at the last level under a total photon cutoff
};
constexpr int pt_vjp_entries(int MD) { return 3 * pt_table_entries(MD) + kPtPos; }

// A lane's constants: A^H (with conj(b) as row 2 MD where it fits), the cutoffs
// of its positions' modes, b where no row serves it.
template <int MD, bool ODD, typename R>
struct VjpPtConst {
  static constexpr int NP = 2 * MD, KS = PtMat<MD, R>::KS;
  static constexpr bool kCol = ODD && NP < kPtPos;   // the pivot as column and row 2 MD
  static constexpr int NCOL = kCol ? NP + 1 : NP;
  PtMat<MD, R> AH;
  int cj[KS];
  cx<R> bl[KS];
  __device__ __forceinline__ void load(const DevPlan& P, const cx<R>* __restrict__ Ai, const cx<R>* __restrict__ bi) {
    const int lane = threadIdx.x & 63, kq = lane >> 4;
    AH.load(Ai, true);
    if (kCol && Mma<R>::row_pos(lane & 15) == NP) {
#pragma unroll
      for (int s = 0; s < KS; ++s)
        if (4 * s + kq < NP) {
          const cx<R> v = ld(bi + 4 * s + kq);
          AH.ar[s] = v.x;
          AH.ai[s] = -v.y;
        }
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      cj[s] = P.CD[min(2 * s + (kq >> 1), MD - 1)];
      bl[s] = ODD && !kCol ? ld(bi + 4 * s + kq) : czero<R>();
    }
  }
};

// A wavefront's sums: Abar (and bbar as a column), or bbar at its positions.
template <int MD, typename R>
struct VjpPtSums {
  MfmaAcc<1> acc;
  double bx[PtMat<MD, R>::KS], by[PtMat<MD, R>::KS];
  __device__ __forceinline__ void zero() {
    mfma_acc_zero(acc);
#pragma unroll
    for (int s = 0; s < PtMat<MD, R>::KS; ++s) bx[s] = by[s] = 0.0;
  }
  // this wavefront's pair table: red[i * NR + l], l = 2 MD the bbar column
  template <bool ODD>
  __device__ __forceinline__ void store(cx<double>* red) const {
    using K = VjpPtConst<MD, ODD, R>;
    constexpr int NP = 2 * MD, NR = NP + 1;
    mfma_acc_store<NP, NR, K::NCOL>(acc, red);
    if (ODD && !K::kCol) {
      const int lane = threadIdx.x & 63, c = lane & 15, kq = lane >> 4;
#pragma unroll
      for (int s = 0; s < K::KS; ++s) {
        double vx = bx[s], vy = by[s];
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
          vx += __shfl_xor(vx, o);
          vy += __shfl_xor(vy, o);
        }
        const int p = 4 * s + kq;
        if (c == 0 && p < NP) red[p * NR + NP] = cmake<double>(vx, vy);
      }
    }
  }
};

// One tile of 16 T points base.. of a level of n points, one wavefront; or (WIDE,
// T = 1) the wavefronts of a workgroup on one tile, bridge K on wavefront K mod
// kWideWaves, which leave the bridges' F0 cotangents and pivot cotangents in LDS
// (`shared`) for the first to finish: the tiles at the start of a level take up to
// 2 MD pivots, 2 us each in one wavefront.
constexpr int kWideWaves = kThreads / 64;
constexpr int wide_entries(int MD) { return (kWideWaves + MD) * 16; }
template <int MD, bool ODD, int T, typename R, bool WIDE = false>
__device__ __forceinline__ void vjp_point_tile(const DevPlan& P, const VjpPtLevel<R>& L,
                                               const VjpPtConst<MD, ODD, R>& C, VjpPtSums<MD, R>& Z,
                                               const uint64_t* mt, int S, int base, int n, cx<R>* turn, int* rows,
                                               cx<R>* shared = nullptr, int wave = 0) {
  static_assert(!WIDE || T == 1, "a workgroup takes one 16-point tile");
  constexpr int NP = 2 * MD, KS = PtMat<MD, R>::KS, SL = 16 * T;
  constexpr bool kCol = VjpPtConst<MD, ODD, R>::kCol;
  constexpr int NCOL = VjpPtConst<MD, ODD, R>::NCOL;
  typedef typename Mma<R>::v4 v4;
  const int lane = threadIdx.x & 63, c = lane & 15, kq = lane >> 4, hk = kq >> 1, side = kq & 1;
  const int pr = c, jr = min(pr >> 1, MD - 1);   // position and mode of the lane's reads x
  {
    const int q = T == 4 ? lane : c;
    pt_rank_rows<MD, T>(P, L.spn, mt, S, min(base + q, n - 1), q, rows);
  }
  wave_sync();
#pragma unroll 1
  for (int t = 0; t < T; ++t) {
    const int r0 = base + 16 * t;
    if (r0 >= n) break;
    const int slot = 16 * t + c;
    const bool live = r0 + c < n;
    const int r = min(r0 + c, n - 1);
    const uint64_t pk = pt_digits<MD, T>(rows, slot);
    // digit and rank of m - 1 at the lane's position 4 s + kq
    auto digit = [&](int s) { return (int)((pk >> (8 * (2 * s + hk))) & 255); };
    auto down = [&](int s) { return rows[min(2 * s + hk, MD - 1) * SL + slot]; };
    const int K0 = pk ? (__ffsll((unsigned long long)pk) - 1) >> 3 : MD;
    const cx<R> d0 = ld(L.d0 + r);
    cx<R> g0 = czero<R>();          // F0 cotangent, in the lanes that hold a position 2 K
    cx<R> gdiag = czero<R>();       // ... from the diagonal pivot's value
    cx<R> yk[KS];                   // cotangents of the bridge pivots F1k(K), at position 2 K
#pragma unroll
    for (int s = 0; s < KS; ++s) yk[s] = czero<R>();

    // reads x of pivot row K (valid columns only: bit 4 s + kq of vm); others
    // read the level's first F0 entry and are discarded
    auto load_x = [&](int K, uint32_t vm, cx<R>(&x)[4]) {
      const bool piv = kCol && pr == NP;
      const bool first = (K < MD && pr == 2 * K) || piv;
      const uint64_t b = L.xp[K * kPtPos + pr];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int q = 16 * t + 4 * s + kq;
        const int m = (int)((pt_digits<MD, T>(rows, q) >> (8 * jr)) & 255);
        const bool ok = ((vm >> (4 * s + kq)) & 1) && pr < NCOL &&
                        (first || ((pr > 2 * K || K == MD) && m > 0));
        const int dn = rows[jr * SL + q];
        const cx<R>* a = global_at<const cx<R>>(b) + (first ? r0 + 4 * s + kq : dn);
        const cx<R> v = ld(ok ? a : L.f0);
        x[s] = cscale(csel(ok, v, czero<R>()), piv ? R(1) : L.sq[m + (first ? 1 : 0)]);
      }
    };
    // D += h conj(x)^T over the tile's 16 points
    auto reduce = [&](const cx<R>(&h)[KS], const cx<R>(&x)[4]) {
#pragma unroll
      for (int s = 0; s < KS; ++s) turn[(4 * s + kq) * kTurn + c] = h[s];
      wave_sync();
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const cx<R> v = turn[pr * kTurn + 4 * s + kq];
        mfma_acc_add<1, R>(Z.acc, 0, v, x[s]);
      }
      wave_sync();
    };
    // b^H h of the point (in its four lanes): row 2 MD of u, or the vector
    // unit's sums, which also add h conj(pivot) to bbar
    auto dot_b = [&](const cx<R>(&h)[KS], const cx<R>& pivot, const v4& re, const v4& im) -> cx<R> {
      if (kCol) {
        const int src = c + 16 * (NP & 3);
        return cmake<R>(__shfl(re[(NP >> 2) & 3], src), __shfl(im[(NP >> 2) & 3], src));
      }
      cx<R> g = czero<R>();
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        cfma_conj(g, C.bl[s], h[s]);
        const double hx = h[s].x, hy = h[s].y, px = pivot.x, py = pivot.y;
        Z.bx[s] += px * hx + py * hy;
        Z.by[s] += px * hy - py * hx;
      }
      g = cadd(g, cmake<R>(__shfl_xor(g.x, 16), __shfl_xor(g.y, 16)));
      return cadd(g, cmake<R>(__shfl_xor(g.x, 32), __shfl_xor(g.y, 32)));
    };

#pragma unroll 1
    for (int K = WIDE ? wave : 0; K < MD; K += WIDE ? kWideWaves : 1) {
      if (__ballot(live && K <= K0) == 0ull) break;
      const int mK = (int)((pk >> (8 * K)) & 255);
      const bool valid = live && K <= K0 && mK <= P.CD[K] - 2;
      const uint64_t vb = __ballot(valid);
      if (vb == 0ull) continue;
      const int up = rows[(MD + K) * SL + slot];
      cx<R> h[KS], x[4];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int p = 4 * s + kq;
        const int two = p == 2 * K ? 1 : 0;
        const bool nxt = p == 2 * K + 1;
        const bool ok = valid && p < NP && p >= 2 * K && digit(s) + two <= C.cj[s] - 2 && (!nxt || L.has_next);
        const cx<R>* a = global_at<const cx<R>>(L.hp[K * kPtPos + p]) + (nxt ? up : r);
        const cx<R> v = ld(ok ? a : L.f0);
        h[s] = cscale(csel(ok, v, czero<R>()), L.isq[digit(s) + 1 + two]);
      }
      load_x(K, (uint32_t)vb & 0xffffu, x);
      cx<R> pv = czero<R>(), gc = czero<R>();
      if (ODD) {
        const bool has_diag_reader = (K > 0) || (mK + 1 <= P.CD[0] - 2);
        const bool lv = valid && has_diag_reader;
        const cx<R>* a = global_at<const cx<R>>(L.hp[MD * kPtPos + 2 * K]) + r;
        const cx<R> g = ld(lv ? a : L.f0);
        gc = csel(lv, g, czero<R>());
        if (!kCol) {
          const cx<R> v = ld(valid ? global_at<const cx<R>>(L.xp[pt_table_entries(MD) + K]) + r : L.f0);
          pv = csel(valid, v, czero<R>());
        }
      }
      v4 re, im;
#pragma unroll
      for (int s = 0; s < 4; ++s) re[s] = im[s] = R(0);
      C.AH.apply(h, re, im);
      // cotangents of the reads
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int p = 4 * s + kq;
        const bool first = p == 2 * K;
        const cx<R> u = cscale(cmake<R>(re[s], im[s]), L.sq[digit(s) + (first ? 1 : 0)]);
        if (first)
          g0 = cadd(g0, csel(valid, u, czero<R>()));
        else if (valid && p < NP && p > 2 * K && digit(s) > 0)
          st(global_at<cx<R>>(L.gp[K * kPtPos + p]) + down(s), u);
      }
      if (ODD) {
        const cx<R> g = cadd(gc, dot_b(h, pv, re, im));
#pragma unroll
        for (int s = 0; s < KS; ++s)
          if (4 * s + kq == 2 * K) {
            yk[s] = g;
            if (WIDE) shared[(kWideWaves + K) * 16 + c] = g;
          }
      }
      reduce(h, x);
    }

    // F0 cotangent: positions 2 K sit in lanes kq = 0 and kq = 2
    g0 = cadd(g0, cmake<R>(__shfl_xor(g0.x, 32), __shfl_xor(g0.y, 32)));
    if (WIDE) {
      if (kq == 0) shared[wave * 16 + c] = g0;
      __syncthreads();
      if (wave != 0) return;
#pragma unroll
      for (int w = 1; w < kWideWaves; ++w) g0 = cadd(g0, shared[w * 16 + c]);
#pragma unroll
      for (int s = 0; s < KS; ++s)
        if (ODD && side == 0 && 2 * s + hk < MD) yk[s] = shared[(kWideWaves + 2 * s + hk) * 16 + c];
    }

    if (ODD) {
      // diagonal pivot
      const bool valid = live && (int)(pk & 255) <= P.CD[0] - 2;
      const uint64_t vb = __ballot(valid);
      if (vb != 0ull) {
        cx<R> h[KS], x[4];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const int p = 4 * s + kq, j = 2 * s + hk;
          const int room = (j == 0 ? P.CD[0] - 2 - side : C.cj[s] - 2) - digit(s);
          const bool ok = valid && p < NP && room >= 0;
          const bool bridge = side == 0 && j <= K0 && digit(s) <= C.cj[s] - 2;   // its cotangent is at hand
          const cx<R>* a = global_at<const cx<R>>(L.hp[MD * kPtPos + p]) + r;
          const cx<R> v = ld(ok && !bridge ? a : L.f0);
          h[s] = cscale(csel(ok, csel(bridge, yk[s], v), czero<R>()), L.isq[digit(s) + 1]);
        }
        load_x(MD, (uint32_t)vb & 0xffffu, x);
        v4 re, im;
#pragma unroll
        for (int s = 0; s < 4; ++s) re[s] = im[s] = R(0);
        C.AH.apply(h, re, im);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const int p = 4 * s + kq;
          if (valid && p < NP && digit(s) > 0)
            st(global_at<cx<R>>(L.gp[MD * kPtPos + p]) + down(s), cscale(cmake<R>(re[s], im[s]), L.sq[digit(s)]));
        }
        cx<R> G0 = czero<R>();
        if (!kCol) {
          const cx<R> v = ld(L.f0 + r);
          G0 = csel(valid, v, G0);
        }
        gdiag = dot_b(h, G0, re, im);
        reduce(h, x);
      }
    }
    if (kq == 0 && live) st(L.g0 + r, cadd(cadd(d0, gdiag), g0));
  }
  wave_sync();   // the rows are rewritten by the next tile
}

}  // namespace fd
