// Shared by the reverse point kernels (vjp_point_units.h) and the reverse block
// kernel (vjp_block.h): the per-level pointer table of the reverse sweep and the
// matrix-core reduction of Abar / bbar.
#pragma once

#include "pt_units.h"

namespace fd {

template <typename R>
struct VjpPtrs {
  const cx<R>* fprev[kMaxFam];  // forward values, level S-1 (store-all)
  const cx<R>* fcur[kMaxFam];   // forward values, level S (fcur[0] = F0)
  cx<R>* gprev[kMaxFam];        // cotangent ring slot of level S-1
  cx<R>* gcur[kMaxFam];         // cotangent ring slot of level S (gcur[0] = F0)
  const cx<R>* gf0nxt;          // F0 cotangents, level S+1
  const cx<R>* d0cur;           // drho in node order, level S
  const int* node;              // node records of level S (Algorithm 2 plans)
  cx<R>* priv;                  // per-workgroup private slots (Algorithm 2 plans)
  int64_t priv_stride;          // entries per slot
};

// Abar / bbar: every reverse step reduces outer products of the target
// cotangents h and the read values x of a pivot application over all of them: D[i][l] = sum h_i conj(x_l), a dense
// contraction over points or block entries, on FP64 MFMA 16x16x4 steps of four
// of them: lane t feeds value t % 16 of number 4 s + t / 16 to both operands and
// keeps D[4 j + t / 16][t % 16], j = 0..3 (the gfx950 output layout, checked on
// the device).  The complex products take three real products (Karatsuba's
// method): P1 = Hr Xr, P2 = Hi Xi, P3 = (Hr + Hi)(Xr - Xi), each summed in its
// own accumulator; the real part is P1 + P2 and the imaginary part (Hi Xr -
// Hr Xi) is P3 - P1 + P2.  Three MFMAs per step instead of four, and three
// independent accumulation chains of one MFMA per step instead of two of
// two.  The hardware fixes the order of accumulation, so the sums are
// reproducible.
typedef double mfma_d4 __attribute__((ext_vector_type(4)));

template <int NT>
struct MfmaAcc {
  mfma_d4 p1[NT], p2[NT], p3[NT];
};

template <int NT>
__device__ __forceinline__ void mfma_acc_zero(MfmaAcc<NT>& a) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    a.p1[t] = mfma_d4{0.0, 0.0, 0.0, 0.0};
    a.p2[t] = mfma_d4{0.0, 0.0, 0.0, 0.0};
    a.p3[t] = mfma_d4{0.0, 0.0, 0.0, 0.0};
  }
}

// One step: h and x are the lane's values, x for column tile t.
template <int NT, typename R>
__device__ __forceinline__ void mfma_acc_add(MfmaAcc<NT>& a, int t, const cx<R>& h, const cx<R>& x) {
  const double hx = h.x, hy = h.y, xx = x.x, xy = x.y;
  a.p1[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(hx, xx, a.p1[t], 0, 0, 0);
  a.p2[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(hy, xy, a.p2[t], 0, 0, 0);
  a.p3[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(hx + hy, xx - xy, a.p3[t], 0, 0, 0);
}

// Writes this lane's accumulated pairs into red[i * NR + l] (a wave's NPD x NR
// pair table); pairs beyond NCOL columns are the caller's (they stay unset).
template <int NPD, int NR, int NCOL>
__device__ __forceinline__ void mfma_acc_store(const MfmaAcc<(NCOL + 15) / 16>& acc, cx<double>* red) {
  constexpr int NT = (NCOL + 15) / 16;
  const int lane = threadIdx.x & 63;
  const int col0 = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int l = 16 * t + col0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = 4 * j + kq;
      if (i < NPD && l < NCOL) {
        const double p1 = acc.p1[t][j], p2 = acc.p2[t][j];
        red[i * NR + l] = cmake<double>(p1 + p2, (acc.p3[t][j] - p1) + p2);
      }
    }
  }
}


constexpr int kTurn = 17;   // row stride of the LDS tile that turns h

// Pointer tables of the reverse step: cotangents of the targets (hp), cotangent
// slots of the reads (gp), forward values of the reads (xp; with PIVOTS, then the
// values of the pivots F1k(K)).
template <int MD, bool ODD, typename R, bool PIVOTS = ODD, typename VP = VjpPtrs<R>>
__device__ __forceinline__ void pt_fill_vjp_pointers(const VP& V, uint64_t* hp, uint64_t* gp, uint64_t* xp) {
  constexpr int NP = 2 * MD;
  for (int t = threadIdx.x; t < pt_table_entries(MD); t += blockDim.x) {
    const int K = t / kPtPos, p = t % kPtPos, j = p >> 1, b = p & 1;
    int ft = -1, fr = -1;   // target (level S, F0: S + 1) and read (level S - 1, F0: S) families
    if (p < NP) {
      if (K == MD) {
        if (ODD) {
          ft = b ? fam_f1b(MD, j) : fam_f1k(j);
          fr = b ? fam_f1k(j) : fam_f1b(MD, j);
        }
      } else if (p == 2 * K) {
        ft = fam_f2(MD, K);
        fr = 0;
      } else if (p == 2 * K + 1) {
        ft = 0;
        fr = fam_f2(MD, K);
      } else if (j > K) {
        ft = b ? fam_1001(MD, K, j) : fam_1010(MD, K, j);
        fr = b ? fam_1010(MD, K, j) : fam_1001(MD, K, j);
      }
    }
    hp[t] = ft < 0 ? 0 : reinterpret_cast<uint64_t>(ft ? V.gcur[ft] : const_cast<cx<R>*>(V.gf0nxt));
    gp[t] = fr < 1 ? 0 : reinterpret_cast<uint64_t>(V.gprev[fr]);
    xp[t] = fr < 0 ? 0 : reinterpret_cast<uint64_t>(fr ? V.fprev[fr] : V.fcur[0]);
    if (ODD && p == NP) xp[t] = reinterpret_cast<uint64_t>(V.fcur[K < MD ? fam_f1k(K) : 0]);   // the pivot's value
  }
  if (PIVOTS)
    for (int K = threadIdx.x; K < MD; K += blockDim.x)
      xp[pt_table_entries(MD) + K] = reinterpret_cast<uint64_t>(V.fcur[fam_f1k(K)]);
}

// One level of the reverse sweep of an Algorithm 2 plan (the block kernel
// for the plan's detected-mode count and block coordinates).
template <typename R>
hipError_t launch_vjp_block_level(const Plan& Pl, const DevPlan& P, const VjpPtrs<R>& Vp, const cx<R>* Ai,
                                  const cx<R>* bi, int S, int nwork, double2* partial, hipStream_t st);

// Its workgroups, each with a reduction slot of its own.
int vjp_block_grid(const Plan& Pl, int nwork);

// The same for a plan with every mode detected (kernels_vjp_point.hip).
template <typename R>
hipError_t launch_vjp_point_level(const Plan& Pl, const DevPlan& P, bool odd, int S, const VjpPtrs<R>& V,
                                  const cx<R>* A, const cx<R>* b, int nwork, double2* partial, hipStream_t st);
int vjp_point_grid(const Plan& Pl, int S);

}  // namespace fd
