// State vectors of pure Gaussian states: psi[n] = <n|psi> for 0 <= n_j < C_j.
//
// The generating function of a pure state has one index per mode (D = M in
// Sec. 2.1), and its scaled Taylor coefficients obey the same recurrence as
// the density matrix's:
//   psi[n] = ( b_i psi[p] + sum_l sqrt(p_l) A_il psi[p - 1_l] ) / sqrt(n_i),
// p = n - 1_i, taken here with i the first mode where n_i > 0.  Targets of
// total photon number S read levels S - 1 and S - 2 only, so the sweep runs
// level by level over the lattice of n (the detected lattice of a plan whose
// modes are all detected: same rank / unrank tables, same level-major
// storage, same output permutation).  With b = 0 the odd levels vanish
// (Sec. 2.4): even levels read level S - 2 alone and odd levels are only
// cleared.
//
// One thread per target; its parent's rank is rdn[i] of the target, its
// parent's own neighbour ranks come from the parent's partial sums (those of
// the target less one up to mode i).
#include <algorithm>
#include <cstring>
#include <vector>

#include "fd_device.h"

namespace fd {

struct StateModes {
  int MD;               // kept modes (cutoff >= 2)
  int mode[kMaxD];      // kept mode k -> caller's mode index
};

// A (symmetrised, (A + A^T)/2, as for density matrices) and b of the kept
// modes into the workspace (MD x MD, then MD), psi at the vacuum = c;
// non-finite inputs set status bit 0, a non-zero b under the b = 0 promise
// status bit 1.
template <typename R>
__global__ __launch_bounds__(64) void k_state_prep(int M, StateModes sm, const cx<R>* __restrict__ A,
                                                   const cx<R>* __restrict__ b, const cx<R>* __restrict__ c,
                                                   cx<R>* __restrict__ Ak, cx<R>* __restrict__ psi0, int check_b_zero,
                                                   int* status) {
  const int MD = sm.MD;
  int bad = 0;
  for (int i = threadIdx.x; i < MD * MD; i += blockDim.x) {
    const cx<R> v = ld(A + (size_t)sm.mode[i / MD] * M + sm.mode[i % MD]);
    const cx<R> w = ld(A + (size_t)sm.mode[i % MD] * M + sm.mode[i / MD]);
    if (!isfinite(v.x) || !isfinite(v.y)) bad |= 1;
    st(Ak + i, cmake<R>(R(0.5) * (v.x + w.x), R(0.5) * (v.y + w.y)));
  }
  for (int i = threadIdx.x; i < M; i += blockDim.x) {
    const cx<R> v = ld(b + i);
    if (!isfinite(v.x) || !isfinite(v.y)) bad |= 1;
    if (check_b_zero && (v.x != R(0) || v.y != R(0))) bad |= 2;
  }
  for (int i = threadIdx.x; i < MD; i += blockDim.x) st(Ak + MD * MD + i, ld(b + sm.mode[i]));
  if (threadIdx.x == 0) {
    const cx<R> cv = ld(c);
    if (!isfinite(cv.x) || !isfinite(cv.y)) bad |= 1;
    st(psi0, cv);
  }
  if (bad) atomicOr(status, bad);
}

// Level S of the sweep (S >= 1; S < 0: none) and, when zlevel >= 0, the
// clearing of level zlevel (an odd level under b = 0).  f0 is psi in level
// order; lvl[S] is the first entry of level S.
template <int MD, bool BZ, typename R>
__global__ __launch_bounds__(kThreads) void k_state_level(DevPlan P, const cx<R>* __restrict__ Ak,
                                                          cx<R>* __restrict__ f0, int S, int zlevel) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<R>* sA = reinterpret_cast<cx<R>*>(smem_raw);   // A (MD x MD) then b (MD)
  const cx<R>* sb = sA + MD * MD;
  R* sq = reinterpret_cast<R*>(sA + MD * MD + MD);
  R* isq = sq + (kMaxCut + 4);
  int* spn = reinterpret_cast<int*>(isq + (kMaxCut + 4));
  const int pnw = P.pnw;
  for (int i = threadIdx.x; i < (MD + 1) * pnw; i += blockDim.x) spn[i] = P.pn[i];
  for (int v = threadIdx.x; v < kMaxCut + 4; v += blockDim.x) {
    sq[v] = sqrt(R(v));
    isq[v] = v ? R(1) / sqrt(R(v)) : R(0);
  }
  for (int i = threadIdx.x; i < MD * MD + MD; i += blockDim.x) sA[i] = ld(Ak + i);
  __syncthreads();
  const int stride = gridDim.x * blockDim.x;
  if (zlevel >= 0) {
    cx<R>* z = f0 + P.lvl[zlevel];
    const int nz = (int)(P.lvl[zlevel + 1] - P.lvl[zlevel]);
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < nz; r += stride) st(z + r, czero<R>());
  }
  if (S < 1) return;
  cx<R>* cur = f0 + P.lvl[S];
  const cx<R>* lv1 = f0 + P.lvl[S - 1];
  const cx<R>* lv2 = S >= 2 ? f0 + P.lvl[S - 2] : f0;
  const int n = (int)(P.lvl[S + 1] - P.lvl[S]);
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
    int m[MD], s[MD + 1], rdn[MD], rup[MD];
    unrank<MD>(spn, pnw, P.CD, S, r, m, s);
    neighbour_ranks<MD>(spn, pnw, s, rdn, rup);
    // first mode with a photon: its index, the parent's rank and n_i
    // (selected with constant indices)
    int i = 0, rp = 0, ni = 1;
    bool found = false;
#pragma unroll
    for (int d = 0; d < MD; ++d)
      if (!found && m[d] > 0) {
        found = true;
        i = d;
        rp = rdn[d];
        ni = m[d];
      }
    // partial sums of the parent p = m - 1_i, then its neighbours at S - 2
    int sp[MD + 1], pdn[MD], pup[MD];
#pragma unroll
    for (int d = 0; d <= MD; ++d) sp[d] = s[d] - (d <= i ? 1 : 0);
    sp[MD] = 0;
    cx<R> acc = czero<R>();
    if (!BZ) cfma(acc, sb[i], ld(lv1 + rp));
    if (S >= 2) {
      neighbour_ranks<MD>(spn, pnw, sp, pdn, pup);
#pragma unroll
      for (int l = 0; l < MD; ++l) {
        const int pl = m[l] - (l == i ? 1 : 0);
        if (pl > 0) cfma(acc, sA[i * MD + l], cscale(ld(lv2 + pdn[l]), sq[pl]));
      }
    }
    st(cur + r, cscale(acc, isq[ni]));
  }
}

// ---------------------------------------------------------------------------
// Derivatives.  The local gradients of Sec. 2.5 (the solutions of its tangent
// recurrences for b and A) have closed forms in the amplitudes:
//   d psi_k / d b_i   = sqrt(k_i) psi_{k - 1_i},
//   d psi_k / d A_il  = 1/2 sqrt(k_i (k_l - [i = l])) psi_{k - 1_i - 1_l},
//   d psi_k / d c     = psi_k / c,
// and every shifted amplitude lies inside the box.  Reverse mode: the
// cotangents bbar_i = sum_k g_k conj(d psi_k / d b_i) (g = dL/dpsi^*, Eqs.
// dL_dB, dL_dA) are weighted dot products of g with shifted copies of psi.
// Forward mode: the tangent along (dA, db, dc) is
//   dpsi_k = (dc / c) psi_k + sum_i db_i sqrt(k_i) psi_{k-1_i}
//          + sum_{i <= l} S_il w_il(k) psi_{k-1_i-1_l},
// S_il = dA_il + dA_li (i < l), dA_ii (i = l), w_il the weight above: the
// directional derivative for the symmetric part of dA, as A enters through
// (A + A^T)/2.
//
// Both kernels number psi (C order, last kept mode fastest) by tiles: the
// trailing modes sp..MD-1 span a tile of T = prod_{d >= sp} C_d entries (at
// most the kernel's tile size) and the leading modes number the tiles, so entry x is
// entry x mod T of tile x / T.  A shifted amplitude of a tile-t entry lies in
// tile t (every mode of the shift trailing), in tile t - 1_i (one leading
// mode i) or in tile t - 1_i - 1_l (two leading modes).  In the forward mode a
// workgroup stages tile t in LDS and serves the terms of the first kind from it, then stages
// tile t - 1_i for each leading i with k_i >= 1 and serves the terms whose
// leading part is 1_i, reading the one amplitude of each two-leading-mode
// term straight from memory.  Each psi entry is so read 1 + (leading modes)
// + (leading pairs) times instead of once per term, and the tile order keeps
// those re-reads in cache: workgroup v runs on XCD v mod 8 and visits tile
// (v mod 8) * ntiles/8 + v / 8, so every XCD walks one contiguous range of
// tiles in order and finds tiles t - 1_i of the faster leading modes in its
// own L2.
// ---------------------------------------------------------------------------
// Tile geometry of each kernel (entries per tile, entries per lane, lanes per
// workgroup): the forward mode stages 64 KB tiles in sixteen-wavefront
// workgroups.
constexpr int kJvpTile = 4096, kJvpEPT = 4, kJvpThreads = kJvpTile / kJvpEPT;
// The reverse mode stages no amplitudes: its tiles only number the entries (and
// at most 2048 of them leave 33 lanes of 64 busy at the worst cutoffs), two
// workgroups of four wavefronts on each CU.
constexpr int kVjpTile = 2048, kVjpGrid = kVjpSlots, kVjpChunk = 8, kVjpUw = kMaxCut;
// Items of a wavefront between two folds of its sums over the lanes (even): a
// lane adds that many terms in a row and the folds go into a compensated sum.  One
// chain over all 256 items of 8 modes cutoff 8 made the gradient's error 6.0e-16 and
// 6.6e-16 on two random states where 512-entry tiles folded one by one had 3.5e-16
// and 4.2e-16; now 2.2e-16 and 3.0e-16, in the same time (912 -> 909 us, amplitudes and
// gradient).
constexpr int kVjpFold = 16;

struct StateTiles {
  int MD, sp, T, ntiles;
  int C[kMaxD], stride[kMaxD];   // kept cutoffs, C-order strides
  double inv_stride[kMaxD], inv_c[kMaxD];
};

static StateTiles state_tiles(const Plan& Pl, int max_tile) {
  StateTiles G;
  std::memset(&G, 0, sizeof(G));
  G.MD = Pl.MD;
  int64_t s = 1;
  for (int d = Pl.MD - 1; d >= 0; --d) {
    G.C[d] = Pl.CD[d];
    G.stride[d] = (int)s;
    G.inv_stride[d] = 1.0 / (double)s;
    G.inv_c[d] = 1.0 / (double)Pl.CD[d];
    s *= Pl.CD[d];
  }
  G.sp = Pl.MD;
  G.T = 1;
  while (G.sp > 0 && G.T * Pl.CD[G.sp - 1] <= max_tile) G.T *= Pl.CD[--G.sp];
  G.ntiles = (int)(s / G.T);
  return G;
}

// Digit (x / stride) mod C of a C-order index x < 2^31: (x + 1/2) / stride
// lies at least 1 / (2 stride) from an integer and the rounded product is off
// by less than (x / stride) 2^-51, so truncation is exact (and so for the mod).
__device__ __forceinline__ int cdigit(int x, int stride, int c, double inv_stride, double inv_c) {
  const int q = (int)((x + 0.5) * inv_stride);
  return q - c * (int)((q + 0.5) * inv_c);
}

// The tile of visit v (see above); in order when the tiles do not split into
// eight equal ranges.
__device__ __forceinline__ int state_tile_of(int ntiles, int v) {
  return (ntiles & 7) ? v : (v & 7) * (ntiles >> 3) + (v >> 3);
}

// Loads tile entries [src, src + T) of this lane (entry f = lane + e * lanes)
// into registers, every load issued before the first is waited on.
template <int NT, int EPT, typename R>
__device__ __forceinline__ void load_lane_entries(cx<R> (&v)[EPT], const cx<R>* __restrict__ src, int T) {
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const int f = threadIdx.x + e * NT;
    v[e] = f < T ? ld(src + f) : czero<R>();
  }
}

// Stages tile entries [src, src + T) in LDS (loads first, then the writes).
template <int NT, int EPT, typename R>
__device__ __forceinline__ void stage_tile(cx<R>* buf, const cx<R>* __restrict__ src, int T) {
  cx<R> v[EPT];
  load_lane_entries<NT, EPT>(v, src, T);
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    const int f = threadIdx.x + e * NT;
    if (f < T) buf[f] = v[e];
  }
}

// acc += (w s) p for a double coefficient s and an amplitude p.
template <typename R>
__device__ __forceinline__ void cmac_w(double& ax, double& ay, double w, double2 s, const cx<R>& p) {
  const double sx = w * s.x, sy = w * s.y;
  ax += sx * (double)p.x - sy * (double)p.y;
  ay += sx * (double)p.y + sy * (double)p.x;
}

template <typename R>
size_t state_jvp_lds_bytes() {
  return (size_t)kJvpTile * sizeof(cx<R>) + (kMaxD * kMaxD + kMaxD) * sizeof(double2) +
         (kMaxCut + 1) * sizeof(double) + kMaxD * sizeof(int);
}

// Forward mode: one workgroup per tile, kJvpEPT entries per lane, the
// tangent accumulated in registers over the tile's phases; the modes are a
// template argument, so the term loops unroll with the strides in scalar
// registers.
template <int MD, typename R>
__global__ __launch_bounds__(kJvpThreads) void k_state_jvp(
    StateTiles G, StateModes sm, int M, const cx<R>* __restrict__ psi, const cx<R>* __restrict__ c,
    const cx<R>* __restrict__ tA, const cx<R>* __restrict__ tb, const cx<R>* __restrict__ tc,
    cx<R>* __restrict__ dpsi) {
  constexpr int MDA = MD > 0 ? MD : 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx<R>* buf = reinterpret_cast<cx<R>*>(smem_raw);
  double2* sS = reinterpret_cast<double2*>(smem_raw + (size_t)kJvpTile * sizeof(cx<R>));   // kMaxD x kMaxD
  double2* sB = sS + kMaxD * kMaxD;
  double* sq = reinterpret_cast<double*>(sB + kMaxD);   // sqrt(0..kMaxCut)
  int* ks = reinterpret_cast<int*>(sq + kMaxCut + 1);  // leading digits of the tile
  const int sp = G.sp, T = G.T;
  for (int v = threadIdx.x; v <= kMaxCut; v += kJvpThreads) sq[v] = sqrt((double)v);
  for (int e = threadIdx.x; e < MD * MD; e += kJvpThreads) {
    const int i = e / MD, l = e % MD;
    const cx<R> a = ld(tA + (size_t)sm.mode[i] * M + sm.mode[l]);
    const cx<R> t = ld(tA + (size_t)sm.mode[l] * M + sm.mode[i]);
    sS[i * kMaxD + l] = i == l ? make_double2(a.x, a.y) : make_double2((double)a.x + t.x, (double)a.y + t.y);
  }
  for (int i = threadIdx.x; i < MD; i += kJvpThreads) {
    const cx<R> v = ld(tb + sm.mode[i]);
    sB[i] = make_double2(v.x, v.y);
  }
  const int x0 = state_tile_of(G.ntiles, blockIdx.x) * T;
  for (int d = threadIdx.x; d < sp; d += kJvpThreads)
    ks[d] = cdigit(x0, G.stride[d], G.C[d], G.inv_stride[d], G.inv_c[d]);
  stage_tile<kJvpThreads, kJvpEPT>(buf, psi + x0, T);
  __syncthreads();
  // dc / c
  const cx<R> cv = ld(c), dv = ld(tc);
  const double n2 = (double)cv.x * cv.x + (double)cv.y * cv.y;
  const double2 r = make_double2(((double)dv.x * cv.x + (double)dv.y * cv.y) / n2,
                                 ((double)dv.y * cv.x - (double)dv.x * cv.y) / n2);
  double ax[kJvpEPT], ay[kJvpEPT];
  // terms inside tile t: dc/c, db_i and the pairs of trailing modes
#pragma unroll
  for (int e = 0; e < kJvpEPT; ++e) {
    const int f = threadIdx.x + e * kJvpThreads;
    ax[e] = 0.0;
    ay[e] = 0.0;
    if (f >= T) continue;
    int k[MDA];
#pragma unroll
    for (int d = 0; d < MD; ++d) k[d] = d >= sp ? cdigit(f, G.stride[d], G.C[d], G.inv_stride[d], G.inv_c[d]) : 0;
    double x = 0.0, y = 0.0;
    cmac_w(x, y, 1.0, r, buf[f]);
#pragma unroll
    for (int i = 0; i < MD; ++i) {
      if (i < sp || k[i] < 1) continue;
      const int fi = f - G.stride[i];
      const double wi = sq[k[i]];
      cmac_w(x, y, wi, sB[i], buf[fi]);
#pragma unroll
      for (int l = i; l < MD; ++l) {
        const int kl = k[l] - (l == i ? 1 : 0);
        if (kl < 1) continue;
        cmac_w(x, y, 0.5 * wi * sq[kl], sS[i * kMaxD + l], buf[fi - G.stride[l]]);
      }
    }
    ax[e] = x;
    ay[e] = y;
  }
  // terms whose leading part is 1_i: tile t - 1_i (uniform over the workgroup)
#pragma unroll
  for (int i = 0; i < MD; ++i) {
    if (i >= sp) continue;
    const int ki = ks[i];
    if (ki < 1) continue;
    const int xs = x0 - G.stride[i];
    __syncthreads();
    stage_tile<kJvpThreads, kJvpEPT>(buf, psi + xs, T);
    __syncthreads();
    const double wi = sq[ki];
#pragma unroll
    for (int e = 0; e < kJvpEPT; ++e) {
      const int f = threadIdx.x + e * kJvpThreads;
      if (f >= T) continue;
      int k[MDA];
#pragma unroll
      for (int d = 0; d < MD; ++d) k[d] = d >= sp ? cdigit(f, G.stride[d], G.C[d], G.inv_stride[d], G.inv_c[d]) : 0;
      double x = ax[e], y = ay[e];
      cmac_w(x, y, wi, sB[i], buf[f]);
#pragma unroll
      for (int l = i + 1; l < MD; ++l) {
        if (l < sp || k[l] < 1) continue;
        cmac_w(x, y, 0.5 * wi * sq[k[l]], sS[i * kMaxD + l], buf[f - G.stride[l]]);
      }
      ax[e] = x;
      ay[e] = y;
    }
    // two leading modes: one amplitude per entry from memory
#pragma unroll
    for (int l = i; l < MD; ++l) {
      if (l >= sp) continue;
      const int kl = ks[l] - (l == i ? 1 : 0);
      if (kl < 1) continue;
      cx<R> p[kJvpEPT];
      load_lane_entries<kJvpThreads, kJvpEPT>(p, psi + (xs - G.stride[l]), T);
      const double w = 0.5 * wi * sq[kl];
      const double2 sc = sS[i * kMaxD + l];
#pragma unroll
      for (int e = 0; e < kJvpEPT; ++e) cmac_w(ax[e], ay[e], w, sc, p[e]);
    }
  }
#pragma unroll
  for (int e = 0; e < kJvpEPT; ++e) {
    const int f = threadIdx.x + e * kJvpThreads;
    if (f < T) st(dpsi + x0 + f, cmake<R>((R)ax[e], (R)ay[e]));
  }
}

// Column of each cotangent: bbar_i (i), Abar_il for i <= l (MD + the upper
// triangle row by row), sum g conj(psi) (last).
__host__ __device__ constexpr int vjp_col_pair(int MD, int i, int l) { return MD + i * MD - i * (i - 1) / 2 + (l - i); }
__host__ __device__ constexpr int vjp_cols(int MD) { return MD + MD * (MD + 1) / 2 + 1; }

// Reverse mode.  With m = k - 1_i the weights of a pair split into one factor
// per mode:
//   Abar_il = 1/2 sum_m u_i(m) conj(v_l(m)),   bbar_i = sum_m u_i(m) conj(psi_m),
//   u_i(m) = sqrt(m_i + 1) g_{m+1_i},  v_l(m) = sqrt(m_l) psi_{m-1_l}
// (zero outside the box), so an entry takes 2 MD shifted loads and scalings for
// its MD (MD + 1) / 2 products, and the lanes keep every sum in registers.  Six to eight modes (28 to 45
// complex sums) are shared by two wavefronts: each has half of the modes as rows i and
// takes every other pair (i, l) between the halves, as u_i v_l or u_l v_i.
//
// What bounds it (8 modes, cutoff 8, c128: 455 us): instructions.  The vector unit
// issues two thirds of the time, 87 M wave instructions in double precision and as
// many others, with two wavefronts per SIMD, which wait a fifth of theirs; the shifts
// along the slower modes miss the L2s, which 1.74 GB leave for 537 MB of psi and g (3.8
// TB/s).  Loading an item only after the products of the one before: 574 us against
// 480; all loads of an item ahead: 28 registers spilled, 827.
// The order of the items does not matter (chunks of 2 to 512: 1045 to 1081 us for the
// call).  The version before staged tiles of psi in LDS and folded each of the
// 45 sums of every tile over the lanes: 620 us.
constexpr int vjp_halves(int MD) { return MD > 5 ? 2 : 1; }
template <int MD>
struct StateVjpSplit {
  static constexpr int half(int i) { return vjp_halves(MD) == 2 && i >= (MD + 1) / 2 ? 1 : 0; }
  // the mode of pair (i, l) that is the row; its half takes the pair
  static constexpr int row(int i, int l) { return half(i) != half(l) && ((i + l) & 1) ? l : i; }
  // columns of half h (the first also has the last column), and its values:
  // real and imaginary parts
  static constexpr int values(int h) {
    int n = h == 0 ? 1 : 0;
    for (int i = 0; i < MD; ++i) {
      if (half(i) == h) ++n;
      for (int l = i; l < MD; ++l)
        if (half(row(i, l)) == h) ++n;
    }
    return 2 * n;
  }
  // fn(column) for each of them, in order
  template <int H, typename F>
  static __device__ __forceinline__ void each(F&& fn) {
    if (H == 0) fn(vjp_cols(MD) - 1);
#pragma unroll
    for (int i = 0; i < MD; ++i) {
      if (half(i) == H) fn(i);
#pragma unroll
      for (int l = i; l < MD; ++l)
        if (half(row(i, l)) == H) fn(vjp_col_pair(MD, i, l));
    }
  }
};

// Sums of N <= 64 values over the lanes of a wavefront.  A step takes values j and
// j + H, H = (N + 1) / 2, of two lanes that differ in one bit: the lane without the
// bit ends with the sum of value j, the other with that of value j + H, so the
// steps halve the number of values (46: 47 exchanges and additions, a butterfly of
// each value 276).  At the end a lane holds one value, fold_index of them.
template <int BIT>
__device__ __forceinline__ double fold_pair(double a, double c) {
  if constexpr (BIT >= 16) {
    // v_permlane32_swap / v_permlane16_swap exchange the upper half (odd rows) of
    // a with the lower half (even rows) of c
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    const u2 ua = __builtin_bit_cast(u2, a), uc = __builtin_bit_cast(u2, c);
    u2 lo, hi;
    if constexpr (BIT == 32) {
      lo = __builtin_amdgcn_permlane32_swap(ua.x, uc.x, false, false);
      hi = __builtin_amdgcn_permlane32_swap(ua.y, uc.y, false, false);
    } else {
      lo = __builtin_amdgcn_permlane16_swap(ua.x, uc.x, false, false);
      hi = __builtin_amdgcn_permlane16_swap(ua.y, uc.y, false, false);
    }
    return __builtin_bit_cast(double, u2{lo.x, hi.x}) + __builtin_bit_cast(double, u2{lo.y, hi.y});
  } else {
    const bool up = (threadIdx.x & BIT) != 0;
    const double keep = up ? c : a, send = up ? a : c;
    // the partner by a data-parallel move: row mirror, half-row mirror, quad swaps
    constexpr int kMove = BIT == 8 ? 0x140 : BIT == 4 ? 0x141 : BIT == 2 ? 0x4e : 0xb1;
    typedef int i2 __attribute__((ext_vector_type(2)));
    const i2 w = __builtin_bit_cast(i2, send);
    const i2 from = {__builtin_amdgcn_update_dpp(0, w.x, kMove, 0xf, 0xf, true),
                     __builtin_amdgcn_update_dpp(0, w.y, kMove, 0xf, 0xf, true)};
    return keep + __builtin_bit_cast(double, from);
  }
}
template <int N, int BIT = 32, int NV>
__device__ __forceinline__ double fold_lanes(double (&v)[NV]) {
  if constexpr (BIT == 0) {
    static_assert(N == 1, "at most 64 values");
    return v[0];
  } else {
    constexpr int H = (N + 1) / 2;
#pragma unroll
    for (int j = 0; j < H; ++j) v[j] = fold_pair<BIT>(v[j], j + H < N ? v[j + H] : 0.0);
    return fold_lanes<H, BIT / 2>(v);
  }
}
// The value that this lane holds after fold_lanes<N>, -1: none.
template <int N, int BIT = 32>
__device__ __forceinline__ int fold_index(int lane) {
  if constexpr (BIT == 0) {
    return 0;
  } else {
    constexpr int H = (N + 1) / 2;
    const int i = fold_index<H, BIT / 2>(lane);
    const int j = i + ((lane & BIT) ? H : 0);
    return i < 0 || j >= N ? -1 : j;
  }
}
__device__ __forceinline__ void add_conj(double& sx, double& sy, double ux, double uy, double vx, double vy) {
  sx += ux * vx + uy * vy;
  sy += uy * vx - ux * vy;
}

// The items of a wavefront (an item: 64 entries of a tile): items j, j + NG ..
// of every chunk c0, c0 + step .. < c1 of kVjpChunk items.
struct StateVjpItems {
  int c0, c1, step, j, items;
};
// An item's entry m and its loads of psi (its own entry where there is no neighbour).
template <int MD, typename R>
struct StateVjpRaw {
  uint64_t pk;   // trailing digits
  int x0, fc;    // tile, entry
  int kd;        // leading digit of mode `lane`
  bool live;
  cx<R> pv[MD > 0 ? MD : 1], p0;
};
// A wavefront's sums over its items, folded over its lanes every kVjpFold items
// (into the lane's `sum` in LDS: value fold_index of the half's columns).  The next item's loads of psi are issued
// before an item's products, those of row i of g after the products of row i (in the
// same registers).  Where an entry lacks one factor of a product, its weight is
// zero; EXACT leaves the product out instead (the value may not be finite).
// sq: the weights of v_l (sqrt(k)), then per mode those of u_i (kVjpUw each).
template <int MD, int HALF, bool EXACT, typename R>
__device__ __forceinline__ void state_vjp_sums(const StateTiles& G, const cx<R>* __restrict__ psi,
                                               const cx<R>* __restrict__ g, const double* sq, const uint64_t* kp,
                                               const StateVjpItems& I, double2* sum) {
  typedef StateVjpSplit<MD> W;
  constexpr int MDA = MD > 0 ? MD : 1, NG = kThreads / 64 / vjp_halves(MD), NV = W::values(HALF);
  const int lane = threadIdx.x & 63, ept = (G.T + 63) >> 6;
  const double* su = sq + kMaxCut + 1;
  struct {
    double x[vjp_cols(MD)], y[vjp_cols(MD)];
  } Z;
#pragma unroll
  for (int p = 0; p < vjp_cols(MD); ++p) Z.x[p] = Z.y[p] = 0.0;
  *sum = make_double2(0.0, 0.0);
  // lane d finds leading digit d of an item's tile
  int dst = 1, dc = 1;
  double dis = 1.0, dic = 1.0;
#pragma unroll
  for (int d = 0; d < MD; ++d)
    if (lane == d) {
      dst = G.stride[d];
      dc = G.C[d];
      dis = G.inv_stride[d];
      dic = G.inv_c[d];
    }
  cx<R> gu[MDA], g0 = czero<R>();
  auto fetch = [&](int q, StateVjpRaw<MD, R>& r) {
    const int tile = q / ept, f = (q - tile * ept) * 64 + lane;
    r.x0 = tile * G.T;
    r.kd = lane < G.sp ? cdigit(r.x0, dst, dc, dis, dic) : 0;
    r.live = f < G.T;
    r.fc = r.live ? f : 0;
    r.pk = kp[r.fc];
    const cx<R>* pp = psi + r.x0;
#pragma unroll
    for (int d = 0; d < MD; ++d) {
      // a leading mode's shift is the same for all lanes, a trailing one's is short
      const bool lead = d < G.sp;
      const int s = G.stride[d], kl = __builtin_amdgcn_readlane(r.kd, d), kt = (int)((r.pk >> (8 * d)) & 255);
      r.pv[d] = ld(pp - (lead && kl > 0 ? s : 0) + (r.fc - (!lead && kt > 0 ? s : 0)));
    }
    r.p0 = ld(pp + r.fc);
  };
  auto fetch_row = [&](int d, const StateVjpRaw<MD, R>& r) {
    const bool lead = d < G.sp;
    const int s = G.stride[d], kl = __builtin_amdgcn_readlane(r.kd, d), kt = (int)((r.pk >> (8 * d)) & 255);
    gu[d] = ld(g + r.x0 + (lead && kl + 1 < G.C[d] ? s : 0) + (r.fc + (!lead && kt + 1 < G.C[d] ? s : 0)));
  };
  auto fetch_rows = [&](const StateVjpRaw<MD, R>& r) {
    if (HALF == 0) g0 = ld(g + r.x0 + r.fc);
#pragma unroll
    for (int d = 0; d < MD; ++d)
      if (W::half(d) == HALF) fetch_row(d, r);
  };
  // the products of item r, then the loads of row after row of item n
  auto add = [&](const StateVjpRaw<MD, R>& r, const StateVjpRaw<MD, R>& n) {
    const double px = (double)r.p0.x, py = (double)r.p0.y;
    int k[MDA];
    double vx[MDA], vy[MDA];
#pragma unroll
    for (int d = 0; d < MD; ++d) {
      k[d] = __builtin_amdgcn_readlane(r.kd, d) + (int)((r.pk >> (8 * d)) & 255);
      const double w = sq[k[d]];
      vx[d] = w * (double)r.pv[d].x;
      vy[d] = w * (double)r.pv[d].y;
    }
    if (HALF == 0) {
      if (r.live) add_conj(Z.x[vjp_cols(MD) - 1], Z.y[vjp_cols(MD) - 1], (double)g0.x, (double)g0.y, px, py);
      g0 = ld(g + n.x0 + n.fc);
    }
#pragma unroll
    for (int i = 0; i < MD; ++i) {
      if (W::half(i) != HALF) continue;
      const double w = r.live ? su[i * kVjpUw + k[i]] : 0.0;
      const bool up = w != 0.0;
      const double ux = w * (double)gu[i].x, uy = w * (double)gu[i].y;
      fetch_row(i, n);
      if (!EXACT || up) add_conj(Z.x[i], Z.y[i], ux, uy, px, py);
#pragma unroll
      for (int l = 0; l < MD; ++l) {
        const int a = i < l ? i : l, b = i < l ? l : i;
        if (W::row(a, b) != i) continue;
        if (!EXACT || (up && k[l] > 0))
          add_conj(Z.x[vjp_col_pair(MD, a, b)], Z.y[vjp_col_pair(MD, a, b)], ux, uy, vx[l], vy[l]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // the lanes' sums since the last fold into sum->x (Knuth's two-sum: sum->y
  // collects what the additions round away)
  auto fold = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    double v[NV];
    int n = 0;
    W::template each<HALF>([&](int p) {
      v[n++] = Z.x[p];
      v[n++] = Z.y[p];
      Z.x[p] = Z.y[p] = 0.0;
    });
    const double t = fold_lanes<NV>(v);
    const double2 a = *sum;
    const double s = a.x + t, b = s - a.x;
    *sum = make_double2(s, a.y + ((a.x - (s - b)) + (t - b)));
    __builtin_amdgcn_sched_barrier(0);
  };
  int c = I.c0, j = I.j;
  // the next item of this wavefront, -1 after the last
  auto next = [&]() -> int {
    if (c >= I.c1 || c * kVjpChunk + j >= I.items) return -1;   // (only the last chunk is short)
    const int q = c * kVjpChunk + j;
    j += NG;
    if (j >= kVjpChunk) {
      j = I.j;
      c += I.step;
    }
    return q;
  };
  StateVjpRaw<MD, R> ra, rb;
  int q = next();
  if (q < 0) return;
  fetch(q, ra);
  fetch_rows(ra);
  for (int left = kVjpFold / 2;; --left) {
    if (left == 0) {
      fold();
      left = kVjpFold / 2;
    }
    const int qb = next();
    fetch(qb >= 0 ? qb : q, rb);
    add(ra, rb);
    if (qb < 0) break;
    q = next();
    fetch(q >= 0 ? q : qb, ra);
    add(rb, ra);
    if (q < 0) break;
  }
  fold();
}

// The sums of one wavefront into red (its row of columns).
template <int MD, int HALF, typename R>
__device__ __forceinline__ void state_vjp_wave(const StateTiles& G, const cx<R>* __restrict__ psi,
                                               const cx<R>* __restrict__ g, const double* sq, const uint64_t* kp,
                                               const StateVjpItems& I, double2* sums, double2* red) {
  typedef StateVjpSplit<MD> W;
  constexpr int NC = vjp_cols(MD), NV = W::values(HALF);
  double2* own = sums + threadIdx.x;
  state_vjp_sums<MD, HALF, false, R>(G, psi, g, sq, kp, I, own);
  if (__ballot(!(fabs(own->x) < __builtin_inf())) != 0ull) state_vjp_sums<MD, HALF, true, R>(G, psi, g, sq, kp, I, own);
  const double sum = own->x + (fabs(own->x) < __builtin_inf() ? own->y : 0.0);
  // this lane's value: real or imaginary part of its column
  const int v = fold_index<NV>(threadIdx.x & 63);
  int n = 0, col = 0;
  W::template each<HALF>([&](int p) { col = (v >> 1) == n++ ? p : col; });
  if (v >= 0) reinterpret_cast<double*>(red + col)[v & 1] = (col >= MD && col < NC - 1 ? 0.5 : 1.0) * sum;
}

// Persistent workgroups (a multiple of 8): workgroup v runs on XCD v mod 8,
// which takes one contiguous eighth of the items in order, so that the shifted
// entries of the faster modes are found in its own L2.  Wavefronts (pairs of
// them where two share the sums) take items in turn; the workgroup adds its
// wavefronts' rows in order into its slot, the final kernel the slots of a column.
template <int MD, typename R>
__global__ __launch_bounds__(kThreads, 2) void k_state_vjp(StateTiles G, const cx<R>* __restrict__ psi,
                                                           const cx<R>* __restrict__ g, double2* __restrict__ slots) {
  constexpr int NC = vjp_cols(MD), NW = kThreads / 64, NG = NW / vjp_halves(MD);
  __shared__ uint64_t kp[kVjpTile];        // trailing digits of a tile's entries, 8 bits per mode
  __shared__ double sq[kMaxCut + 1 + (MD > 0 ? MD : 1) * kVjpUw];
  __shared__ double2 red[NW * NC], sums[kThreads];
  for (int v = threadIdx.x; v <= kMaxCut; v += kThreads) sq[v] = sqrt((double)v);
#pragma unroll
  for (int d = 0; d < MD; ++d)
    for (int v = threadIdx.x; v < kVjpUw; v += kThreads)
      sq[kMaxCut + 1 + d * kVjpUw + v] = v + 1 < G.C[d] ? sqrt(v + 1.0) : 0.0;
  for (int p = threadIdx.x; p < NW * NC; p += kThreads) red[p] = make_double2(0.0, 0.0);
  for (int f = threadIdx.x; f < G.T; f += kThreads) {
    uint64_t p = 0;
#pragma unroll
    for (int d = 0; d < MD; ++d)
      if (d >= G.sp) p |= (uint64_t)cdigit(f, G.stride[d], G.C[d], G.inv_stride[d], G.inv_c[d]) << (8 * d);
    kp[f] = p;
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int items = G.ntiles * ((G.T + 63) >> 6), chunks = (items + kVjpChunk - 1) / kVjpChunk;
  const int per = (chunks + 7) >> 3, xcd = blockIdx.x & 7;
  const StateVjpItems I{xcd * per + (int)(blockIdx.x >> 3), min((xcd + 1) * per, chunks), (int)(gridDim.x >> 3),
                        wave / vjp_halves(MD), items};
  if (vjp_halves(MD) == 1 || (wave & 1) == 0)
    state_vjp_wave<MD, 0, R>(G, psi, g, sq, kp, I, sums, red + wave * NC);
  else
    state_vjp_wave<MD, vjp_halves(MD) - 1, R>(G, psi, g, sq, kp, I, sums, red + wave * NC);
  __syncthreads();
  for (int p = threadIdx.x; p < NC; p += kThreads) {
    double sx = 0.0, sy = 0.0;
    for (int wv = 0; wv < NW; ++wv) {
      sx += red[wv * NC + p].x;
      sy += red[wv * NC + p].y;
    }
    slots[(size_t)blockIdx.x * NC + p] = make_double2(sx, sy);
  }
}

// One workgroup per caller entry of dA (M x M), db (M), dc: the slots of its
// column added in order (zero for modes with cutoff 1), Abar mirrored.
struct StateVjpMap {
  int M, MD, ncol, nslots;
  int mode[kMaxD];
};

template <typename R>
__global__ __launch_bounds__(kThreads) void k_state_vjp_final(StateVjpMap m, const double2* __restrict__ slots,
                                                              const cx<R>* __restrict__ c, cx<R>* dA, cx<R>* db,
                                                              cx<R>* dc) {
  __shared__ double2 red[kThreads];
  const int e = blockIdx.x, M = m.M, MD = m.MD;
  int col = -1;
  if (e < M * M) {
    int ki = -1, kl = -1;
    for (int d = 0; d < MD; ++d) {
      if (m.mode[d] == e / M) ki = d;
      if (m.mode[d] == e % M) kl = d;
    }
    if (ki >= 0 && kl >= 0) {
      const int a = min(ki, kl), bb = max(ki, kl);
      col = MD + a * MD - a * (a - 1) / 2 + (bb - a);   // columns: bbar (MD), then the upper triangle row by row
    }
  } else if (e < M * M + M) {
    for (int d = 0; d < MD; ++d)
      if (m.mode[d] == e - M * M) col = d;
  } else {
    col = m.ncol - 1;
  }
  double sx = 0.0, sy = 0.0;
  if (col >= 0)
    for (int s = threadIdx.x; s < m.nslots; s += blockDim.x) {
      sx += slots[(size_t)s * m.ncol + col].x;
      sy += slots[(size_t)s * m.ncol + col].y;
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
  double2 t = red[0];
  if (e < M * M) {
    st(dA + e, cmake<R>((R)t.x, (R)t.y));
  } else if (e < M * M + M) {
    st(db + (e - M * M), cmake<R>((R)t.x, (R)t.y));
  } else {
    // cbar = sum g conj(psi / c) = (sum g conj(psi)) / conj(c)
    const cx<R> cv = ld(c);
    const double cr = (double)cv.x, ci = (double)cv.y, n2 = cr * cr + ci * ci;
    st(dc, cmake<R>((R)((t.x * cr - t.y * ci) / n2), (R)((t.y * cr + t.x * ci) / n2)));
  }
}

template <int MD, typename R>
static void launch_state_jvp(const StateTiles& G, const StateModes& sm, int M, const void* psi, const void* c,
                             const void* dA, const void* db, const void* dc, void* dpsi, hipStream_t st) {
  const size_t shm = state_jvp_lds_bytes<R>();
  if (shm > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_state_jvp<MD, R>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  hipLaunchKernelGGL((k_state_jvp<MD, R>), dim3((unsigned)G.ntiles), dim3(kJvpThreads), shm, st, G, sm, M,
                     static_cast<const cx<R>*>(psi), static_cast<const cx<R>*>(c), static_cast<const cx<R>*>(dA),
                     static_cast<const cx<R>*>(db), static_cast<const cx<R>*>(dc), static_cast<cx<R>*>(dpsi));
}

template <typename R>
static hipError_t launch_state_jvp_md(const StateTiles& G, const StateModes& sm, int M, const void* psi,
                                      const void* c, const void* dA, const void* db, const void* dc, void* dpsi,
                                      hipStream_t st) {
  switch (G.MD) {
    case 0: launch_state_jvp<0, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    case 1: launch_state_jvp<1, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    case 2: launch_state_jvp<2, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    case 3: launch_state_jvp<3, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    case 4: launch_state_jvp<4, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    case 5: launch_state_jvp<5, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    case 6: launch_state_jvp<6, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    case 7: launch_state_jvp<7, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    case 8: launch_state_jvp<8, R>(G, sm, M, psi, c, dA, db, dc, dpsi, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t run_state_jvp(const Plan& Pl, const void* c, const void* psi, const void* dA, const void* db, const void* dc,
                         void* dpsi, hipStream_t st) {
  StateModes sm;
  std::memset(&sm, 0, sizeof(sm));
  sm.MD = Pl.MD;
  for (int k = 0; k < Pl.MD; ++k) sm.mode[k] = Pl.dmodes[k];
  const StateTiles G = state_tiles(Pl, kJvpTile);
  KTimer kt(Pl, KK_FWD_LEVEL, st);
  if (Pl.dt == FD_C64) return launch_state_jvp_md<float>(G, sm, Pl.M, psi, c, dA, db, dc, dpsi, st);
  return launch_state_jvp_md<double>(G, sm, Pl.M, psi, c, dA, db, dc, dpsi, st);
}

template <typename R>
static hipError_t run_state_vjp_t(const Plan& Pl, const void* c, const void* psi, const void* g, void* dA, void* db,
                                  void* dc, void* ws, hipStream_t st) {
  const int MD = Pl.MD, ncol = MD + MD * (MD + 1) / 2 + 1;
  double2* slots = static_cast<double2*>(ws);
  const StateTiles G = state_tiles(Pl, kVjpTile);
  // at most kVjpGrid workgroups (a multiple of 8), one slot each
  static_assert(kVjpGrid % 8 == 0, "one share of the items per XCD");
  const int64_t items = (int64_t)G.ntiles * ((G.T + 63) / 64);
  const int grid = (int)std::min<int64_t>((items + 8 * kVjpChunk - 1) / (8 * kVjpChunk) * 8, kVjpGrid);
  {
    KTimer kt(Pl, KK_VJP_LEVEL, st);
#define FD_STATE_VJP(MDV)                                                                                  \
  case MDV:                                                                                                \
    hipLaunchKernelGGL((k_state_vjp<MDV, R>), dim3((unsigned)grid), dim3(kThreads), 0, st, G,              \
                       static_cast<const cx<R>*>(psi), static_cast<const cx<R>*>(g), slots);               \
    break;
    switch (MD) {
      FD_STATE_VJP(0)
      FD_STATE_VJP(1)
      FD_STATE_VJP(2)
      FD_STATE_VJP(3)
      FD_STATE_VJP(4)
      FD_STATE_VJP(5)
      FD_STATE_VJP(6)
      FD_STATE_VJP(7)
      FD_STATE_VJP(8)
      default: return hipErrorInvalidValue;
    }
#undef FD_STATE_VJP
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  StateVjpMap m;
  std::memset(&m, 0, sizeof(m));
  m.M = Pl.M;
  m.MD = MD;
  m.ncol = ncol;
  m.nslots = grid;
  for (int d = 0; d < MD; ++d) m.mode[d] = Pl.dmodes[d];
  KTimer kt(Pl, KK_VJP_FINAL, st);
  hipLaunchKernelGGL((k_state_vjp_final<R>), dim3(Pl.M * Pl.M + Pl.M + 1), dim3(kThreads), 0, st, m, slots,
                     static_cast<const cx<R>*>(c), static_cast<cx<R>*>(dA), static_cast<cx<R>*>(db),
                     static_cast<cx<R>*>(dc));
  return hipGetLastError();
}

hipError_t run_state_vjp(const Plan& Pl, const void* c, const void* psi, const void* g, void* dA, void* db, void* dc,
                         void* ws, hipStream_t st) {
  if (Pl.dt == FD_C64) return run_state_vjp_t<float>(Pl, c, psi, g, dA, db, dc, ws, st);
  return run_state_vjp_t<double>(Pl, c, psi, g, dA, db, dc, ws, st);
}

template <typename R>
static hipError_t run_state_fwd_t(const Plan& Pl, bool bz, const void* A, const void* b, const void* c, void* psi,
                                  void* ws, hipStream_t st) {
  const size_t eb = sizeof(cx<R>);
  cx<R>* f0 = static_cast<cx<R>*>(ws);
  cx<R>* Ak = reinterpret_cast<cx<R>*>(static_cast<char*>(ws) + (((size_t)Pl.nodes_total * eb + 255) & ~size_t(255)));
  StateModes sm;
  std::memset(&sm, 0, sizeof(sm));
  sm.MD = Pl.MD;
  for (int k = 0; k < Pl.MD; ++k) sm.mode[k] = Pl.dmodes[k];
  {
    KTimer kt(Pl, KK_PREP, st);
    hipLaunchKernelGGL((k_state_prep<R>), dim3(1), dim3(64), 0, st, Pl.M, sm, static_cast<const cx<R>*>(A),
                       static_cast<const cx<R>*>(b), static_cast<const cx<R>*>(c), Ak, f0, bz ? 1 : 0,
                       Pl.d_status);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const DevPlan P = make_devplan(Pl, !bz);
  const size_t shm = (size_t)(Pl.MD * Pl.MD + Pl.MD) * eb + 2 * (kMaxCut + 4) * sizeof(R) +
                     (size_t)(Pl.MD + 1) * (Pl.smax + 3) * sizeof(int);
  auto count = [&](int S) { return S >= 0 && S <= Pl.smax ? Pl.lvl[S + 1] - Pl.lvl[S] : int64_t(0); };
  auto launch = [&](int S, int zl) -> hipError_t {
    const int64_t work = std::max(count(S), count(zl));
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((work + kThreads - 1) / kThreads, 65536));
    KTimer kt(Pl, KK_FWD_LEVEL, st);
#define FD_STATE_LEVEL(MDV)                                                                                \
  case MDV:                                                                                                \
    if (bz)                                                                                                \
      hipLaunchKernelGGL((k_state_level<MDV, true, R>), dim3(grid), dim3(kThreads), shm, st, P, Ak, f0, S, zl); \
    else                                                                                                   \
      hipLaunchKernelGGL((k_state_level<MDV, false, R>), dim3(grid), dim3(kThreads), shm, st, P, Ak, f0, S, zl); \
    break;
    switch (Pl.MD) {
      FD_STATE_LEVEL(1)
      FD_STATE_LEVEL(2)
      FD_STATE_LEVEL(3)
      FD_STATE_LEVEL(4)
      FD_STATE_LEVEL(5)
      FD_STATE_LEVEL(6)
      FD_STATE_LEVEL(7)
      FD_STATE_LEVEL(8)
      default: return hipErrorInvalidValue;
    }
#undef FD_STATE_LEVEL
    return hipGetLastError();
  };
  for (int S = 1; S <= Pl.smax && Pl.MD > 0; ++S) {
    if (bz && (S & 1)) continue;   // odd level: cleared with the next even one
    if ((e = launch(S, bz ? S - 1 : -1)) != hipSuccess) return e;
  }
  if (bz && Pl.MD > 0 && (Pl.smax & 1))
    if ((e = launch(-1, Pl.smax)) != hipSuccess) return e;
  return launch_out_perm(Pl, f0, psi, st);
}

hipError_t run_state_fwd(const Plan& Pl, bool b_zero, const void* A, const void* b, const void* c, void* psi, void* ws,
                         hipStream_t st) {
  if (Pl.dt == FD_C64) return run_state_fwd_t<float>(Pl, b_zero, A, b, c, psi, ws, st);
  return run_state_fwd_t<double>(Pl, b_zero, A, b, c, psi, ws, st);
}

}  // namespace fd
