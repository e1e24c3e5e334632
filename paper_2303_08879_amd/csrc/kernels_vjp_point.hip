// Reverse level kernels of plans with every mode detected (Algorithm 1): one
// launch per level, the points in tiles of 16 columns on the matrix cores.
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
// What bounds it: 48 bytes per computed amplitude.  With one point per lane the
// two 16-vectors and the reduction's staging held 202 VGPRs + 17 KB of LDS per
// wavefront (two wavefronts per SIMD, 60 % of their cycles waiting).
#include <algorithm>

#include "pt_units.h"
#include "vjp_common.h"

namespace fd {

// Two wavefronts per SIMD asked for: the compiler then keeps the MFMA operands
// and results out of the accumulation registers (8 modes, b = 0: 200 -> 184).
template <int MD, bool ODD, int T, typename R>
__global__ __launch_bounds__(kThreads, 2) void k_vjp_point(DevPlan P, VjpPtrs<R> V, const uint64_t* __restrict__ mt,
                                                        const cx<R>* __restrict__ Ai, const cx<R>* __restrict__ bi,
                                                        int S, int nwork, double2* __restrict__ partial) {
  constexpr int NP = 2 * MD, NR = NP + 1, NPAIR = NP * NR, KS = PtMat<MD, R>::KS, SL = 16 * T;
  typedef typename Mma<R>::v4 v4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  R* sq = reinterpret_cast<R*>(smem_raw);
  const R* isq = sq + (kMaxCut + 4);
  uint64_t* hp = reinterpret_cast<uint64_t*>(sq + 2 * (kMaxCut + 4));
  uint64_t* gp = hp + pt_table_entries(MD);
  uint64_t* xp = gp + pt_table_entries(MD);
  cx<R>* turn = reinterpret_cast<cx<R>*>(xp + pt_table_entries(MD));
  int* rows = reinterpret_cast<int*>(turn + (kThreads / 64) * kPtPos * kTurn);
  int* spn = rows + (kThreads / 64) * pt_row_ints(MD, T);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c = lane & 15, kq = lane >> 4, hk = kq >> 1, side = kq & 1;
  turn += wave * kPtPos * kTurn;
  rows += wave * pt_row_ints(MD, T);
  pt_load_tables<R>(P, MD, sq, spn);
  pt_fill_vjp_pointers<MD, ODD, R>(V, hp, gp, xp);
  constexpr bool kCol = ODD && NP < kPtPos;   // the pivot as column and row 2 MD
  constexpr int NCOL = kCol ? NP + 1 : NP;
  PtMat<MD, R> AH;
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
  int cj[KS];
  cx<R> bl[KS];   // b at the lane's positions, where no column serves it
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    cj[s] = P.CD[min(2 * s + hk, MD - 1)];
    bl[s] = ODD && !kCol ? ld(bi + 4 * s + kq) : czero<R>();
  }
  __syncthreads();
  const cx<R>* f0 = V.fcur[0];
  const bool has_next = V.gf0nxt != nullptr;   // false at the last level under a total photon cutoff
  MfmaAcc<1> acc;
  mfma_acc_zero(acc);
  double bx[KS], by[KS];   // bbar at this lane's positions, over its points
#pragma unroll
  for (int s = 0; s < KS; ++s) bx[s] = by[s] = 0.0;
  const int pr = lane & 15, jr = min(pr >> 1, MD - 1);   // position and mode of the lane's reads x

  const int stride = gridDim.x * (kThreads / 64) * SL;
  for (int base = (blockIdx.x * (kThreads / 64) + wave) * SL; base < nwork; base += stride) {
    {
      const int q = T == 4 ? lane : c;
      pt_rank_rows<MD, T>(P, spn, mt, S, min(base + q, nwork - 1), q, rows);
    }
    wave_sync();
#pragma unroll 1
    for (int t = 0; t < T; ++t) {
      const int r0 = base + 16 * t;
      if (r0 >= nwork) break;
      const int slot = 16 * t + c;
      const bool live = r0 + c < nwork;
      const int r = min(r0 + c, nwork - 1);
      const uint64_t pk = pt_digits<MD, T>(rows, slot);
      // digit and rank of m - 1 at the lane's position 4 s + kq
      auto digit = [&](int s) { return (int)((pk >> (8 * (2 * s + hk))) & 255); };
      auto down = [&](int s) { return rows[min(2 * s + hk, MD - 1) * SL + slot]; };
      const int K0 = pk ? (__ffsll((unsigned long long)pk) - 1) >> 3 : MD;
      const cx<R> d0 = ld(V.d0cur + r);
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
        const uint64_t b = xp[K * kPtPos + pr];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int q = 16 * t + 4 * s + kq;
          const int m = (int)((pt_digits<MD, T>(rows, q) >> (8 * jr)) & 255);
          const bool ok = ((vm >> (4 * s + kq)) & 1) && pr < NCOL &&
                          (first || ((pr > 2 * K || K == MD) && m > 0));
          const cx<R> v = ld(ok ? global_at<const cx<R>>(b) + (first ? r0 + 4 * s + kq : rows[jr * SL + q]) : f0);
          x[s] = cscale(csel(ok, v, czero<R>()), piv ? R(1) : sq[m + (first ? 1 : 0)]);
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
          mfma_acc_add<1, R>(acc, 0, v, x[s]);
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
          cfma_conj(g, bl[s], h[s]);
          const double hx = h[s].x, hy = h[s].y, px = pivot.x, py = pivot.y;
          bx[s] += px * hx + py * hy;
          by[s] += px * hy - py * hx;
        }
        g = cadd(g, cmake<R>(__shfl_xor(g.x, 16), __shfl_xor(g.y, 16)));
        return cadd(g, cmake<R>(__shfl_xor(g.x, 32), __shfl_xor(g.y, 32)));
      };

#pragma unroll 1
      for (int K = 0; K < MD; ++K) {
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
          const bool ok = valid && p < NP && p >= 2 * K && digit(s) + two <= cj[s] - 2 && (!nxt || has_next);
          const cx<R> v = ld(ok ? global_at<const cx<R>>(hp[K * kPtPos + p]) + (nxt ? up : r) : f0);
          h[s] = cscale(csel(ok, v, czero<R>()), isq[digit(s) + 1 + two]);
        }
        load_x(K, (uint32_t)vb & 0xffffu, x);
        cx<R> pv = czero<R>(), gc = czero<R>();
        if (ODD) {
          const bool has_diag_reader = (K > 0) || (mK + 1 <= P.CD[0] - 2);
          const bool lv = valid && has_diag_reader;
          const cx<R> g = ld(lv ? V.gcur[fam_f1k(K)] + r : f0);
          gc = csel(lv, g, czero<R>());
          if (!kCol) {
            const cx<R> v = ld(valid ? V.fcur[fam_f1k(K)] + r : f0);
            pv = csel(valid, v, czero<R>());
          }
        }
        v4 re, im;
#pragma unroll
        for (int s = 0; s < 4; ++s) re[s] = im[s] = R(0);
        AH.apply(h, re, im);
        // cotangents of the reads
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const int p = 4 * s + kq;
          const bool first = p == 2 * K;
          const cx<R> u = cscale(cmake<R>(re[s], im[s]), sq[digit(s) + (first ? 1 : 0)]);
          if (first)
            g0 = cadd(g0, csel(valid, u, czero<R>()));
          else if (valid && p < NP && p > 2 * K && digit(s) > 0)
            st(global_at<cx<R>>(gp[K * kPtPos + p]) + down(s), u);
        }
        if (ODD) {
          const cx<R> g = cadd(gc, dot_b(h, pv, re, im));
#pragma unroll
          for (int s = 0; s < KS; ++s)
            if (4 * s + kq == 2 * K) yk[s] = g;
        }
        reduce(h, x);
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
            const int room = (j == 0 ? P.CD[0] - 2 - side : cj[s] - 2) - digit(s);
            const bool ok = valid && p < NP && room >= 0;
            const bool bridge = side == 0 && j <= K0 && digit(s) <= cj[s] - 2;   // its cotangent is at hand
            const cx<R> v = ld(ok && !bridge ? global_at<const cx<R>>(hp[MD * kPtPos + p]) + r : f0);
            h[s] = cscale(csel(ok, csel(bridge, yk[s], v), czero<R>()), isq[digit(s) + 1]);
          }
          load_x(MD, (uint32_t)vb & 0xffffu, x);
          v4 re, im;
#pragma unroll
          for (int s = 0; s < 4; ++s) re[s] = im[s] = R(0);
          AH.apply(h, re, im);
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            const int p = 4 * s + kq;
            if (valid && p < NP && digit(s) > 0)
              st(global_at<cx<R>>(gp[MD * kPtPos + p]) + down(s), cscale(cmake<R>(re[s], im[s]), sq[digit(s)]));
          }
          cx<R> G0 = czero<R>();
          if (!kCol) {
            const cx<R> v = ld(f0 + r);
            G0 = csel(valid, v, G0);
          }
          gdiag = dot_b(h, G0, re, im);
          reduce(h, x);
        }
      }
      // F0 cotangent: positions 2 K sit in lanes kq = 0 and kq = 2
      const cx<R> o = cmake<R>(__shfl_xor(g0.x, 32), __shfl_xor(g0.y, 32));
      if (kq == 0 && live) st(V.gcur[0] + r, cadd(cadd(d0, gdiag), cadd(g0, o)));
    }
    wave_sync();   // the rows are rewritten by the next tile
  }
  // fold the wavefronts' pair tables (fixed order) into this workgroup's slot
  cx<double>* red = reinterpret_cast<cx<double>*>(smem_raw);
  __syncthreads();
  mfma_acc_store<NP, NR, NCOL>(acc, red + (size_t)wave * NPAIR);
  if (ODD && !kCol) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      double vx = bx[s], vy = by[s];
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        vx += __shfl_xor(vx, o);
        vy += __shfl_xor(vy, o);
      }
      const int p = 4 * s + kq;
      if (c == 0 && p < NP) red[(size_t)wave * NPAIR + p * NR + NP] = cmake<double>(vx, vy);
    }
  }
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

int vjp_point_grid(int nwork) {
  const int per = kThreads / 64 * 16 * (nwork >= kPointTileMin ? 4 : 1);
  return std::min((nwork + per - 1) / per, kPartialSlots - 1);
}

template <int T, typename R>
static hipError_t launch_t(const Plan& Pl, const DevPlan& P, bool odd, int S, const VjpPtrs<R>& V, const cx<R>* A,
                           const cx<R>* b, int nwork, double2* partial, hipStream_t st) {
  const size_t shm =
      std::max(pt_lds_bytes(Pl, T, kThreads / 64, 3) + (size_t)(kThreads / 64) * kPtPos * kTurn * sizeof(cx<R>),
               (size_t)(kThreads / 64) * 2 * Pl.MD * (2 * Pl.MD + 1) * sizeof(cx<double>));
  const uint64_t* mt = Pl.d_mtab ? Pl.d_mtab + Pl.lvl[S] : nullptr;
  const int grid = vjp_point_grid(nwork);
#define FD_VJP_POINT(MDV)                                                                                          \
  case MDV:                                                                                                        \
    if (odd)                                                                                                       \
      hipLaunchKernelGGL((k_vjp_point<MDV, true, T, R>), dim3(grid), dim3(kThreads), shm, st, P, V, mt, A, b, S,   \
                         nwork, partial);                                                                          \
    else                                                                                                           \
      hipLaunchKernelGGL((k_vjp_point<MDV, false, T, R>), dim3(grid), dim3(kThreads), shm, st, P, V, mt, A, b, S,  \
                         nwork, partial);                                                                          \
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
