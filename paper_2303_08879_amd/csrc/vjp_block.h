// Reverse sweep of Algorithm 2 plans: the block kernel and its per-level
// launch, compiled in four translation units (precision, detected modes 1-4
// and 5-8); the fills and the sweep driver are in kernels_vjp.hip.
#pragma once

#include <algorithm>

#include "vjp_common.h"

namespace fd {

// ---------------------------------------------------------------------------
// Algorithm 2 reverse step.  One workgroup of four or eight wavefronts (vjp_waves)
// per (lattice point, chunk of rows of the first undetected coordinate).  The undetected
// neighbour terms make the cotangent of a pivot entry pull from the entry one
// row below, so a chunk recomputes the target cotangents of two rows past its
// own (bridge pivots: the rows its diagonal pivot needs; diagonal pivot: one
// row), without storing them.
// The entries of a chunk are the columns of the products, 16 per wavefront and
// step as in the point kernel: u = [A b]^H h gives the cotangents of the undetected
// neighbours (rows 0..NQ-1, kept in LDS: the entry below picks them up), of the
// detected reads (stored to their only reader's slot) and of the pivot (the last
// row); D += h conj(x)^T over the chunk's own entries gives Abar and bbar.  The read
// values come from memory in the operand's layout, the undetected neighbours' from
// the pivot's own row (a cache hit).  Everything but the entry's index is
// uniform over a (lattice point, bridge), so a lane keeps one pointer per position.
// What bounds it: 48 bytes per computed amplitude.  One entry per lane held two
// full vectors and staged them in LDS, 76 KB per workgroup; it moved 1.9 TB/s.
// ST: the neighbour terms, b terms and own rows in the workgroup's private
// slot in global memory (blocks whose rows do not fit the LDS); the
// __syncthreads between phases are workgroup-scope fences.
// ---------------------------------------------------------------------------
// Wavefronts per SIMD that the registers are cut to.  From 16 positions on the
// instances in double precision hold 330 to 460 registers, and one wavefront that
// keeps them beats two that spill 200 (reverse sweeps: an undetected mode of cutoff
// 10 behind eight detected of cutoff 3 1664 -> 1058 us, cutoff 16 behind eight of
// cutoff 2 733 -> 514); in single precision two with 60-110 spilled are no slower
// (898 -> 876; one without: 886).
template <int MD, int NQ, typename R>
constexpr int kVjpBlockSimd = NQ + 2 * MD >= 16 && sizeof(R) == 8 ? 1 : 2;

template <int MD, int NQ, typename R, bool ST>
__global__ __launch_bounds__(64 * vjp_waves(MD, NQ), (kVjpBlockSimd<MD, NQ, R>)) void k_vjp_block(DevPlan P, VjpPtrs<R> V, const cx<R>* __restrict__ Ai,
                                                                 const cx<R>* __restrict__ bi, int S, int nwork,
                                                                 ChunkGeo G, double2* __restrict__ partial) {
  constexpr int NPD = 2 * MD, NPOS = NQ + NPD, NR = NPOS + 1, NPAIR = NPD * NR;
  // 16 positions: the pivot's row and column would take a second tile each, so
  // they are formed on the vector unit (cutoff 20 behind seven detected of cutoff 3
  // 1124 -> 965 us per reverse sweep, in single precision 847 -> 701)
  constexpr bool kPiv = NPOS == 16;
  constexpr int NM = kPiv ? NPOS : NR;   // rows of u and columns of D that are products
  constexpr int KS = (NPD + 3) / 4;      // steps over the targets
  constexpr int NT = (NM + 15) / 16;     // tiles of rows of u, and of columns of D
  constexpr int WV = vjp_waves(MD, NQ);
  // one undetected mode with five and six detected in double precision, seven in single:
  // 10-25 registers over the two wavefronts' 256, unless what a lane derives from its
  // position is formed anew for every pivot and the scales are looked up where they are
  // used (five of cutoff 8 behind cutoff 30: 7920 -> 7790 us, six of cutoff 4 behind
  // 12: 739 -> 667); the other instances lose 3-10 % by it
  constexpr bool kTight = NQ == 2 && (sizeof(R) == 8 ? KS > 2 && kVjpBlockSimd<MD, NQ, R> == 2 : kPiv);
  typedef typename Mma<R>::v4 v4;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int B = P.B, R0 = G.R0, RC = G.RC;
  const int nrow1 = (RC + 1) * R0, nrow2 = (RC + 2) * R0;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 15, kq = lane >> 4;
  R* sq = reinterpret_cast<R*>(smem_raw);
  const R* isq = sq + (kMaxCut + 4);
  uint64_t* hp = reinterpret_cast<uint64_t*>(sq + 2 * (kMaxCut + 4));
  uint64_t* gp = hp + pt_table_entries(MD);
  uint64_t* xp = gp + pt_table_entries(MD);
  cx<R>* turn = reinterpret_cast<cx<R>*>(xp + pt_table_entries(MD));   // waves x NPD x kTurn
  cx<R>* rows = turn + WV * NPD * kTurn;
  turn += wave * NPD * kTurn;
  cx<R>* gpk = V.priv + (size_t)blockIdx.x * V.priv_stride;   // bridge pivots' cotangents, MD x rows [k0, k1+1)
  cx<R>* gbv = ST ? gpk + (size_t)MD * nrow1 : rows;          // b^H h of the bridge, rows [k0, k1+1)
  cx<R>* g0a = gbv + nrow1;                                   // F0 cotangent, own rows
  cx<R>* qv = g0a + RC * R0;                                  // neighbour terms, NQ x rows [k0, k1+2)
  {
    const R* t = reinterpret_cast<const R*>(P.sqt);
    for (int i = threadIdx.x; i < 2 * (kMaxCut + 4); i += blockDim.x) sq[i] = t[i];
  }
  pt_fill_vjp_pointers<MD, true, R, false>(V, hp, gp, xp);
  // [A b]^H: row l = 16 t + row, column i = 4 s + kq
  R ar[NT][KS], ai[NT][KS];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int l = 16 * t + Mma<R>::row_pos(c), i = 4 * s + kq;
      const bool in = l < NM && i < NPD;
      const cx<R> v = ld(!in ? Ai : l < NPOS ? Ai + (NQ + i) * NPOS + l : bi + NQ + i);
      ar[t][s] = in ? v.x : R(0);
      ai[t][s] = in ? -v.y : R(0);
    }
  // the undetected coordinate of a lane whose read is a neighbour (columns l < NQ)
  const int ql = min(c, NQ - 1);
  const int us = P.ustride[ql], ud = P.udims[ql];
  // single precision splits entries below 65536 exactly: (e + 1/2) / us lies at
  // least 1 / (2 us) from an integer, the product is off by less than e 2^-23 / us
  const float ui = 1.0f / (float)us, di = 1.0f / (float)ud;
  int cj[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) cj[s] = P.CD[min((4 * s + kq) >> 1, MD - 1)];
  // the cotangent that a row is added to is read before the products (three
  // undetected modes, double precision: 446 -> 411 us and 520 -> 505 per reverse sweep)
  // or, in fewer registers, after them
  constexpr bool kAhead = NQ == 6 && sizeof(R) == 8 && NT == 1 && !kPiv;
  MfmaAcc<NT> acc;
  mfma_acc_zero(acc);
  constexpr int KV = kPiv ? KS : 1;
  cx<R> bl[KV];            // b at the lane's positions, and its sums of bbar there
  double bx[KV], by[KV];
#pragma unroll
  for (int s = 0; s < KV; ++s) {
    bl[s] = kPiv && 4 * s + kq < NPD ? ld(bi + NQ + 4 * s + kq) : czero<R>();
    bx[s] = by[s] = 0.0;
  }
  __syncthreads();

  for (int w = blockIdx.x; w < nwork * G.nchunks; w += gridDim.x) {
    const int r = w / G.nchunks, ch = w - r * G.nchunks;
    const int k0 = ch * RC, k1 = min(G.C0, k0 + RC);
    const int e0 = k0 * R0, e1 = k1 * R0;                          // own entries
    const int eb1 = min(G.C0, k1 + 1) * R0, eq1 = min(G.C0, k1 + 2) * R0;
    const int nrec = V.node[(size_t)r * kNodeStride + min(lane, kNodeStride - 1)];
    auto m_of = [&](int j) { return __shfl(nrec, j); };
    auto down = [&](int j) { return __shfl(nrec, MD + j); };
    const int m0 = __builtin_amdgcn_readlane(nrec, 0);
    const size_t rB = (size_t)r * B;
    if (m0 > P.CD[0] - 2) {   // no pivot here (uniform)
      for (int e = e0 + threadIdx.x; e < e1; e += blockDim.x) st(V.gcur[0] + rB + e, ld(V.d0cur + rB + e));
      continue;
    }
    int K0 = MD;
#pragma unroll
    for (int d = MD - 1; d >= 0; --d)
      if (__builtin_amdgcn_readlane(nrec, d) > 0) K0 = d;

    // sum over the undetected neighbours above entry e of their terms
    auto neighbours = [&](int e, cx<R> v) -> cx<R> {
      int rem = e;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int k = ucoord(P, rem, q);
        rem -= k * P.ustride[q];
        if (k + 1 < P.udims[q]) v = cadd(v, cscale(qv[(size_t)q * nrow2 + (e - e0) + P.ustride[q]], sq[k + 1]));
      }
      return v;
    };

    // the pivots: K < MD the bridges d(m) + 1_ket(K), then (K = MD) the diagonal
#pragma unroll 1
    for (int K = 0; K <= MD; ++K) {
      const bool diag = K == MD;
      if (!diag && K > K0) continue;
      const int mK = diag ? 0 : __builtin_amdgcn_readlane(nrec, K);
      if (!diag && mK > P.CD[K] - 2) continue;   // uniform
      const int up = diag ? 0 : __builtin_amdgcn_readlane(nrec, 2 * MD + K);
      const int ee = diag ? eb1 : eq1;                        // entries [e0, ee) of the targets
      const cx<R>* pv = V.fcur[diag ? 0 : fam_f1k(K)] + rB;   // the pivot's values
      // targets: pointer and scale of each of the lane's positions
      int kv = kq, cv = c;
      if (kTight) asm volatile("" : "+v"(kv), "+v"(cv));   // (what follows is not moved out of the loops)
      // (kTight: scales as 8-bit indexes into the square-root tables)
      const cx<R>* hptr[KS];
      R hw[KS];
      uint32_t hi = 0, hv = 0;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const int p = 4 * s + kv, j = min(p >> 1, MD - 1), side = p & 1;
        const int mj = m_of(j);
        const int two = p == 2 * K ? 1 : 0;
        const int room = cj[s] - 2 - mj - (diag && j == 0 ? side : two);
        const bool ok = p < NPD && room >= 0 && (diag || p >= 2 * K);
        const bool bridge = diag && side == 0 && j <= K0 && mj <= cj[s] - 2;   // its cotangent is at hand
        const cx<R>* t = global_at<const cx<R>>(hp[K * kPtPos + p]) + (p == 2 * K + 1 ? (size_t)up * B : rB);
        t = bridge ? gpk + (size_t)j * nrow1 - e0 : t;
        hptr[s] = ok ? t : pv;
        hw[s] = isq[mj + 1 + two];
        hi |= (uint32_t)(kMaxCut + 4 + mj + 1 + two) << (8 * s);
        hv |= (ok ? 1u : 0u) << s;
      }
      // read values: columns l = 16 t + c
      const cx<R>* xptr[NT];
      R xw[NT];
      uint32_t xi = 0, xv = 0;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int l = 16 * t + cv, p = l - NQ, pc = min(max(p, 0), NPD - 1), j = pc >> 1;
        const int mj = m_of(j), dn = down(j);
        const bool first = p == 2 * K, det = p >= 0 && p < NPD;
        const bool ok = l < NM && (!det || first || ((diag || p > 2 * K) && mj > 0));
        xptr[t] = !ok || !det ? pv : global_at<const cx<R>>(xp[K * kPtPos + pc]) + (first ? rB : (size_t)dn * B);
        xw[t] = sq[det ? mj + (first ? 1 : 0) : 1];
        xi |= (uint32_t)(det ? mj + (first ? 1 : 0) : 1) << (8 * t);
        xv |= (ok ? 1u : 0u) << t;
      }
      // where the rows of u go: the cotangents of the detected reads to their
      // slots in memory; the neighbour terms, the b terms and the F0 cotangent
      // (added to) to the unit's rows, at offset loff, entries below lend
      cx<R>* gptr[NT * 4];
      R gw[NT * 4];
      uint32_t gi[NT] = {};
      int loff[NT * 4], lend[NT * 4];
      uint32_t gv = 0, lsum = 0;
#pragma unroll
      for (int t = 0; t < NT * 4; ++t) {
        const int l = 4 * t + kv, p = l - NQ, pc = min(max(p, 0), NPD - 1), j = pc >> 1;
        const int mj = m_of(j), dn = down(j);
        const bool det = p >= 0 && p < NPD, first = p == 2 * K;
        const bool ok = det && (diag || p > 2 * K) && mj > 0;
        gptr[t] = global_at<cx<R>>(gp[K * kPtPos + pc]) + (ok ? (size_t)dn * B : 0);
        gw[t] = sq[det ? first ? mK + 1 : mj : 1];
        gi[t / 4] |= (uint32_t)(det ? first ? mK + 1 : mj : 1) << (8 * (t % 4));
        gv |= (ok ? 1u : 0u) << t;
        const bool nb = l < NQ, piv = l == NPOS;
        loff[t] = nb ? (2 * RC + 1) * R0 + l * nrow2 : piv && !diag ? 0 : nrow1;
        lend[t] = nb ? ee : piv && !diag ? eb1 : piv || (det && first) ? e1 : e0;
        lsum |= (piv ? diag : first) ? 1u << t : 0u;
      }
      // the row of u that the F0 cotangent adds up, and whether this lane holds it
      const int srow = diag ? NPOS : NQ + 2 * K;
      const bool sums = kq == (srow & 3);
      // read column t of entry ex: neighbour columns read the entry one step
      // down in their coordinate, with its square root as weight
      auto xcol = [&](int t, int ex, int* at, R* wt) -> bool {
        bool ok = ex < e1 && ((xv >> t) & 1);
        *at = ex;
        *wt = kTight ? sq[(xi >> (8 * t)) & 255] : xw[t];
        if (t == 0) {
          const int q = (int)(((float)ex + 0.5f) * ui);
          const int kc = q - ud * (int)(((float)q + 0.5f) * di);
          const bool nb = c < NQ;
          const R wq = sq[kc];
          ok = ok && (!nb || kc > 0);
          *at = nb ? ex - us : ex;
          *wt = nb ? wq : *wt;
        }
        *at = ok ? *at : e0;
        return ok;
      };
      // the tile's loads, unconditional and unscaled: issued one tile ahead
      // (a load waited on within the tile's work would wait for them all), but
      // for the few reads beyond column 16, which go out before the next tile's
      auto load_x = [&](int t, int eb, cx<R>(&x)[4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          int at;
          R wt;
          (void)xcol(t, eb + 4 * s + kq, &at, &wt);
          x[s] = ld(xptr[t] + at);
        }
      };
      auto issue = [&](int eb, cx<R>(&h)[KS], cx<R>(&x)[4], cx<R>& d0, cx<R>& pval) {
        const int e = eb + c;
        if (kPiv) pval = ld(pv + min(e, e1 - 1));
        if (K == 0) d0 = ld(V.d0cur + rB + min(e, e1 - 1));
#pragma unroll
        for (int s = 0; s < KS; ++s) h[s] = ld(hptr[s] + (e < ee ? e : e0));
        if (eb < e1) load_x(0, eb, x);
      };
      cx<R> hn[KS], xn[4], dn = czero<R>(), pn = czero<R>();
      if (e0 + 16 * wave < ee) issue(e0 + 16 * wave, hn, xn, dn, pn);
#pragma unroll 1
      for (int eb = e0 + 16 * wave; eb < ee; eb += 16 * WV) {
        const int e = eb + c, le = e - e0;
        const bool live = e < ee, own = e < e1;
        const bool any_own = eb < e1;   // uniform
        cx<R> h[KS], x[NT][4];
#pragma unroll
        for (int s = 0; s < KS; ++s) h[s] = hn[s];
#pragma unroll
        for (int s = 0; s < 4; ++s) x[0][s] = xn[s];
        if (any_own) {
#pragma unroll
          for (int t = 1; t < NT; ++t) load_x(t, eb, x[t]);
        }
        const cx<R> d0 = dn, pval = pn;
        if (eb + 16 * WV < ee) issue(eb + 16 * WV, hn, xn, dn, pn);
        cx<R> was = czero<R>();
        if (kAhead && sums && own) was = K == 0 ? d0 : g0a[le];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const bool ok = live && ((hv >> s) & 1);
          h[s] = cscale(csel(ok, h[s], czero<R>()), kTight ? sq[(hi >> (8 * s)) & 255] : hw[s]);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          v4 re, im;
#pragma unroll
          for (int s = 0; s < 4; ++s) re[s] = im[s] = R(0);
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            re = Mma<R>::mma(ar[t][s], h[s].x, re);
            im = Mma<R>::mma(ar[t][s], h[s].y, im);
            re = Mma<R>::mma(ai[t][s], -h[s].y, re);
            im = Mma<R>::mma(ai[t][s], h[s].x, im);
          }
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int i = 4 * t + s;
            if (4 * i >= NM) continue;   // no such rows
            const cx<R> u = cscale(cmake<R>(re[s], im[s]), kTight ? sq[(gi[t] >> (8 * s)) & 255] : gw[i]);
            cx<R>* slot = gbv + loff[i] + le;
            if (e < lend[i]) {
              if (kAhead) {
                *slot = i == (srow >> 2) ? cadd(u, was) : u;
              } else {
                was = *slot;
                was = csel(K == 0, d0, was);
                *slot = cadd(u, csel((lsum >> i) & 1, was, czero<R>()));
              }
            }
            if (own && ((gv >> i) & 1)) st(gptr[i] + e, u);
          }
        }
        if (kPiv) {
          // the pivot's row, b^H h, in the four lanes of an entry, and its column of D
          cx<R> g = czero<R>();
#pragma unroll
          for (int s = 0; s < KV; ++s) {
            cfma_conj(g, bl[s], h[s]);
            const cx<R> ho = csel(own, h[s], czero<R>());
            const double hx = ho.x, hy = ho.y, px = pval.x, py = pval.y;
            bx[s] += px * hx + py * hy;
            by[s] += px * hy - py * hx;
          }
          g = cadd(g, cmake<R>(__shfl_xor(g.x, 16), __shfl_xor(g.y, 16)));
          g = cadd(g, cmake<R>(__shfl_xor(g.x, 32), __shfl_xor(g.y, 32)));
          if (kq == 0) {
            if (diag && own) g0a[le] = cadd(g, g0a[le]);
            if (!diag && e < eb1) gbv[le] = g;
          }
        }
        if (any_own) {
          // D over the own entries (h of the others as zero)
#pragma unroll
          for (int s = 0; s < KS; ++s)
            if (4 * s + kq < NPD) turn[(4 * s + kq) * kTurn + c] = csel(own, h[s], czero<R>());
          wave_sync();
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const cx<R> ht = turn[min(c, NPD - 1) * kTurn + 4 * s + kq];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              int at;
              R wt;
              const bool ok = xcol(t, eb + 4 * s + kq, &at, &wt);
              mfma_acc_add<NT, R>(acc, t, ht, cscale(csel(ok, x[t][s], czero<R>()), wt));
            }
          }
          wave_sync();
        }
      }
      __syncthreads();
      if (!diag) {
        // total cotangent of the bridge pivot block F1k(K)(m), rows [k0, k1+1)
        const bool has_diag_reader = (K > 0) || (m0 + 1 <= P.CD[0] - 2);
        const cx<R>* gc = V.gcur[fam_f1k(K)] + rB;
        for (int e = e0 + threadIdx.x; e < eb1; e += blockDim.x) {
          cx<R> v = gbv[e - e0];
          if (has_diag_reader) v = cadd(v, ld(gc + e));
          gpk[(size_t)K * nrow1 + (e - e0)] = neighbours(e, v);
        }
        __syncthreads();
      }
    }
    for (int e = e0 + threadIdx.x; e < e1; e += blockDim.x) st(V.gcur[0] + rB + e, neighbours(e, g0a[e - e0]));
    __syncthreads();
  }
  // fold the waves' pair tables (in wave order) into this block's slot
  cx<double>* red = reinterpret_cast<cx<double>*>(smem_raw);
  __syncthreads();
  mfma_acc_store<NPD, NR, NM>(acc, red + (size_t)wave * NPAIR);
  if (kPiv) {
#pragma unroll
    for (int s = 0; s < KV; ++s) {
      double vx = bx[s], vy = by[s];
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        vx += __shfl_xor(vx, o);
        vy += __shfl_xor(vy, o);
      }
      const int p = 4 * s + kq;
      if (c == 0 && p < NPD) red[(size_t)wave * NPAIR + p * NR + NPOS] = cmake<double>(vx, vy);
    }
  }
  __syncthreads();
  double2* slot = partial + (size_t)blockIdx.x * (NPOS * NR);
  for (int p = threadIdx.x; p < NPAIR; p += blockDim.x) {
    const int i = p / NR, l = p - (p / NR) * NR;
    const int q = (NQ + i) * NR + l;
    double sx = 0.0, sy = 0.0;
    for (int wv = 0; wv < WV; ++wv) {
      sx += red[(size_t)wv * NPAIR + p].x;
      sy += red[(size_t)wv * NPAIR + p].y;
    }
    const double2 v = slot[q];
    slot[q] = make_double2(v.x + sx, v.y + sy);
  }
}

template <int MD, int NQ, typename R, bool ST>
static void launch_vjp_block_k(size_t shm, int grid, hipStream_t st, const DevPlan& P, const VjpPtrs<R>& Vp,
                               const cx<R>* Ai, const cx<R>* bi, int S, int nwork, const ChunkGeo& G,
                               double2* partial) {
  if (shm > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_vjp_block<MD, NQ, R, ST>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  hipLaunchKernelGGL((k_vjp_block<MD, NQ, R, ST>), dim3(grid), dim3(64 * vjp_waves(MD, NQ)), shm, st, P, Vp, Ai, bi, S, nwork,
                     G, partial);
}

// Detected modes LO..LO + 3.
template <typename R, int LO>
hipError_t launch_vjp_block_range(const Plan& Pl, const DevPlan& P, const VjpPtrs<R>& Vp, const cx<R>* Ai,
                                  const cx<R>* bi, int S, int nwork, double2* partial, hipStream_t st) {
  const int MD = Pl.MD;
  // as in the forward sweep: shorter row chunks on levels with few units
  const ChunkGeo G = vjp_geo(Pl, nwork);
  const size_t shm = vjp_lds_bytes_for(Pl, G);
  if (shm > kMaxLds) return hipErrorInvalidConfiguration;   // rejected before the sweep
  const int grid = vjp_block_grid(Pl, nwork);
#define FD_VJP_BLOCK_NQ(MDV, NQV)                                                                       \
  if (Pl.st_vjp)                                                                                   \
    launch_vjp_block_k<MDV, NQV, R, true>(shm, grid, st, P, Vp, Ai, bi, S, nwork, G, partial); \
  else                                                                                             \
    launch_vjp_block_k<MDV, NQV, R, false>(shm, grid, st, P, Vp, Ai, bi, S, nwork, G, partial);
#define FD_VJP_BLOCK(MDV)        \
  case LO + MDV:                 \
    if (Pl.nq == 2) {            \
      FD_VJP_BLOCK_NQ(LO + MDV, 2)    \
    } else if (Pl.nq == 4) {     \
      FD_VJP_BLOCK_NQ(LO + MDV, 4)    \
    } else {                     \
      FD_VJP_BLOCK_NQ(LO + MDV, 6)    \
    }                            \
    break;
  switch (MD) {
    FD_VJP_BLOCK(0)
    FD_VJP_BLOCK(1)
    FD_VJP_BLOCK(2)
    FD_VJP_BLOCK(3)
    default:
      return hipErrorInvalidValue;
  }
#undef FD_VJP_BLOCK
#undef FD_VJP_BLOCK_NQ
  return hipSuccess;
}

}  // namespace fd
