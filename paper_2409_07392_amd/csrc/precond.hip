// Block-diagonal preconditioner of Definition 1 / eq. 12:
//   P_k = shift I_d + sum_i omega_i h_ik (1 - h_ik) x_i x_i^T,   k = 0..c-1,
// followed by an FP64 Cholesky factorisation P_k = L_k L_k^T and the explicit
// inverse P_k^-1 = L_k^-T L_k^-1 used by the PCG apply.
//
// The c weighted Gram matrices are one GEMM over rows, classes against (a, b)
// pairs, with both operands formed from H, omega and X while they are staged;
// slices of rows are reduced afterwards in FP64 in a fixed order.
#include <algorithm>
#include <climits>
#include <cstdlib>
#include <type_traits>
#include <utility>
#include <vector>

#include "common.h"

namespace firal {

// Weighted Gram matrices as one GEMM: P[k][(a, b)] = sum_i u_ik w_i,(a,b) with u_ik =
// omega_i h_ik (1 - h_ik) (classes: the M dimension) and w_i,(a,b) = x_ia x_ib (pairs: the N
// dimension), k over the rows.  A pair tile is a 16 x BR block of (a, b) in or below the
// diagonal band; each row stage stages u for the class tile and the tile's 16 + BR x values
// in LDS, and the MFMA B operand is formed as x_a x_b when it is read.  Four waves in a
// WC x (4 / WC) arrangement (classes x pairs), each CMW x PNW blocks of 16 x 16: with few
// classes (c <= 16) all four waves sit along the pairs.
// Rows per stage: 32 for FP32 (half the barriers of 16-row stages: 2.13 -> 2.04 s for the 1000
// blocks of 384 x 384 over 1.28M rows), 16 for FP64 (32 would need 83 KB of LDS, leaving one
// workgroup per CU).
template <typename T> constexpr int kSyrkTK = sizeof(T) == 4 ? 32 : 16;
__constant__ double kSyrkUnitWeight = 1.0;   // the row weight when none is given

// L is the storage type of X and H (FP32 rows feed the FP64 Gram of the Round step).
template <typename T, typename L, int CMW, int PNW, int WC>
__global__ __launch_bounds__(256, 2) void k_syrk(const L* __restrict__ X, const L* __restrict__ H,
                                                 const double* __restrict__ omega, int64_t N,
                                                 int d, int c, const int32_t* __restrict__ tiles,
                                                 int ntiles, int nct, int64_t rows_per_split,
                                                 T* __restrict__ part) {
  constexpr int TK = kSyrkTK<T>;   // rows per stage
  constexpr int WP = 4 / WC;
  constexpr int TC = 16 * CMW * WC, TP = 16 * PNW * WP, BR = TP / 16;
  constexpr int SU = TC + 16;
  constexpr int EU = TC * TK / 256;
  __shared__ __align__(16) T Us[2][TK][SU];
  __shared__ T Xa[2][TK][17];
  __shared__ T Xb[2][TK][BR + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, g = lane >> 4;
  // logical tile: class tile fastest, then pair tile, then row split
  const int64_t lid = blockIdx.x;
  const int cls_t = (int)(lid % nct);
  const int64_t rest = lid / nct;
  const int pt = (int)(rest % ntiles);
  const int sp = (int)(rest / ntiles);
  const int c0 = cls_t * TC;
  const int a0 = 16 * tiles[2 * pt], b0 = BR * tiles[2 * pt + 1];
  const int64_t rb = (int64_t)sp * rows_per_split;
  const int64_t re = rb + rows_per_split < N ? rb + rows_per_split : N;
  const int wc = (wave / WP) * 16 * CMW, wp = (wave % WP) * 16 * PNW;

  typedef Mfma16<T> M;
  typename M::acc acc[CMW][PNW];
#pragma unroll
  for (int i = 0; i < CMW; ++i)
#pragma unroll
    for (int j = 0; j < PNW; ++j) acc[i][j] = M::zero();

  // staging: u for (row k, class); the 16 x_a and BR x_b values of each row k
  const int ucls = tid % TC, uk = tid / TC;
  constexpr int KU = 256 / TC;
  const bool uvalid = c0 + ucls < c;
  constexpr int XW = 16 + BR, XE = TK * XW, NX = (XE + 255) / 256;
  int xk[NX], xj[NX];
  bool xon[NX], xvalid[NX];
#pragma unroll
  for (int i = 0; i < NX; ++i) {
    const int e = tid + 256 * i;
    xon[i] = e < XE;
    xk[i] = e / XW;
    xj[i] = e % XW;
    const int col = xj[i] < 16 ? a0 + xj[i] : b0 + (xj[i] - 16);
    xvalid[i] = xon[i] && col < d;
    xj[i] = xvalid[i] ? col : 0;   // column of X to load (when valid)
  }
  // The loads read rows clamped into the split (rb is a row of it whenever there is a stage) and
  // classes and columns clamped into the arrays; u = w h (1 - h) is formed and the values outside
  // the tile are zeroed when the stage is stored, so no loaded value is consumed before the
  // current stage's MFMAs.
  L rh[EU], rx[NX];   // as stored (converted to T when staged)
  double rw[EU];
  const int uc = uvalid ? c0 + ucls : 0;
  const double* wsrc = omega ? omega : &kSyrkUnitWeight;
  auto load = [&](int kt) {
    const int64_t r0 = rb + (int64_t)kt * TK;
#pragma unroll
    for (int i = 0; i < EU; ++i) {
      const int64_t r = r0 + uk + KU * i;
      rh[i] = H[(r < re ? r : rb) * c + uc];
    }
#pragma unroll
    for (int i = 0; i < EU; ++i) {   // without weights every row reads the one weight 1
      const int64_t r = r0 + uk + KU * i;
      rw[i] = wsrc[omega ? (r < re ? r : rb) : 0];
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int64_t r = r0 + xk[i];
      rx[i] = X[(r < re ? r : rb) * d + xj[i]];
    }
  };
  auto store = [&](int buf, int kt) {
    const int64_t r0 = rb + (int64_t)kt * TK;
#pragma unroll
    for (int i = 0; i < EU; ++i) {
      const int64_t r = r0 + uk + KU * i;
      const T h = (T)rh[i];
      const T u = (T)rw[i] * h * (T(1) - h);
      Us[buf][uk + KU * i][ucls] = r < re && uvalid ? u : T(0);
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      // every thread stores (threads without an element write the unread pad column of Xa), so
      // that the compiler keeps each load in the load phase rather than sinking it here
      const int e = tid + 256 * i, j = e % XW;
      const int64_t r = r0 + xk[i];
      const T v = r < re && xvalid[i] ? (T)rx[i] : T(0);
      T* dst = !xon[i] ? &Xa[buf][0][16] : (j < 16 ? &Xa[buf][xk[i]][j] : &Xb[buf][xk[i]][j - 16]);
      *dst = v;
    }
  };

  const int64_t nrows = re > rb ? re - rb : 0;
  const int nk = (int)((nrows + TK - 1) / TK);
  if (nk > 0) {
    load(0);
    store(0, 0);
  }
  __syncthreads();
  // this lane's pairs in the B operand: (a_local, b_local) of column wp + 16 j + li
  int pa[PNW], pb[PNW];
#pragma unroll
  for (int j = 0; j < PNW; ++j) {
    const int pp = wp + 16 * j + li;
    pa[j] = pp / BR;
    pb[j] = pp % BR;
  }
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    load(kt + 1);   // past the last stage every row is out of range (stored as zero, never read)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < TK / 4; ++q) {
      const int k = 4 * q + g;
      T av[CMW], bv[PNW];
#pragma unroll
      for (int i = 0; i < CMW; ++i) av[i] = Us[buf][k][wc + 16 * i + li];
#pragma unroll
      for (int j = 0; j < PNW; ++j) bv[j] = Xa[buf][k][pa[j]] * Xb[buf][k][pb[j]];
#pragma unroll
      for (int i = 0; i < CMW; ++i)
#pragma unroll
        for (int j = 0; j < PNW; ++j) acc[i][j] = M::run(av[i], bv[j], acc[i][j]);
    }
    __builtin_amdgcn_sched_barrier(0);
    store(buf ^ 1, kt + 1);
    __syncthreads();
  }

  T* out = part + (int64_t)sp * c * d * d;
#pragma unroll
  for (int i = 0; i < CMW; ++i)
#pragma unroll
    for (int j = 0; j < PNW; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = c0 + wc + 16 * i + M::row(g, v);
        const int a = a0 + pa[j], b = b0 + pb[j];
        if (k < c && a < d && b < d && b <= a) out[((int64_t)k * d + a) * d + b] = acc[i][j][v];
      }
}

// The same Gram GEMM with the four waves along the pairs, for FP32-storage contexts with c > 64
// classes and d a multiple of 4: a pair tile of 16 a x 16 b columns against 128 classes, wave w
// taking a columns 4 w .. 4 w + 3 against all 16 b columns and all classes of the tile, so a pair
// product x_a x_b is formed once per workgroup and feeds CMW class blocks.  Stages of 32 rows;
// u = omega h (1 - h) is staged as [class][row] and the tile's x values as FP32 [column][row], so
// each lane reads its rows of a class or a column as 16-byte vectors.
//   FP32 (BF3 false): v_mfma_f32_16x16x4f32, the 16-row groups of a stage in the k order of the
//     wide products (lane group g takes rows 4 g + q of the group for instruction q, so one
//     16-byte read of u or x feeds four instructions).
//   bf16x3 (BF3 true, the opt-in of bf16x3 contexts): u split into hi/lo bf16 planes when staged;
//     each lane forms the products for its 8 rows (8 g .. 8 g + 7) in FP32 and splits them in
//     registers; three 16x16x32 bf16 MFMAs per block (hi hi + hi lo + lo hi).
constexpr int kSwTK = 32;                        // rows per stage (the bf16 MFMA's k)
constexpr int kSwXS = kSwTK + 4;                 // LDS row of a staged x column, floats
template <bool BF3> constexpr int kSwUS = BF3 ? kSwTK + 8 : kSwTK + 4;   // LDS row of u
template <int CMW, bool BF3>
__global__ __launch_bounds__(256, 2) void k_syrkw(const float* __restrict__ X,
                                                  const float* __restrict__ H,
                                                  const double* __restrict__ omega, int64_t N,
                                                  int d, int c, const int32_t* __restrict__ tiles,
                                                  int ntiles, int nct, int64_t rows_per_split,
                                                  float* __restrict__ part) {
  constexpr int TC = 16 * CMW, NQ = TC / 64, US = kSwUS<BF3>;
  static_assert(TC % 64 == 0, "u staging: 64 classes per quarter of the workgroup");
  typedef typename std::conditional<BF3, __bf16, float>::type UT;
  __shared__ __align__(16) UT Us[BF3 ? 2 : 1][2][TC][US];   // [hi, lo] or [u]
  __shared__ __align__(16) float XaT[2][16][kSwXS];
  __shared__ __align__(16) float XbT[2][16][kSwXS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int li = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t lid = blockIdx.x;
  const int cls_t = (int)(lid % nct);
  const int64_t rest = lid / nct;
  const int pt = (int)(rest % ntiles);
  const int sp = (int)(rest / ntiles);
  const int c0 = cls_t * TC;
  const int a0 = 16 * tiles[2 * pt], b0 = 16 * tiles[2 * pt + 1];
  const int64_t rb = (int64_t)sp * rows_per_split;
  const int64_t re = rb + rows_per_split < N ? rb + rows_per_split : N;

  f32x4 acc[CMW][4];
#pragma unroll
  for (int i = 0; i < CMW; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // staging: u of classes (tid % 64) + 64 q for the 8 rows 8 wave .. 8 wave + 7 of the stage
  // (the row weights are the same for a whole wave); one 4-float x vector per thread: row
  // tid / 8, columns a0 + 4 (tid % 8) (tid % 8 < 4) or b0 + 4 (tid % 8 - 4)
  int ucls[NQ];
  bool uvalid[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    ucls[q] = (tid & 63) + 64 * q;
    uvalid[q] = c0 + ucls[q] < c;
  }
  const int xr = tid >> 3, xp = tid & 7;
  const int xcol = xp < 4 ? a0 + 4 * xp : b0 + 4 * (xp - 4);
  const bool xvalid = xcol < d;   // d and the column a multiple of 4: all four in or all out
  const double* wsrc = omega ? omega : &kSyrkUnitWeight;
  float rh[NQ][8];
  double rw[8];
  f32x4 rx;
  // loads read rows clamped into the split and columns clamped into the arrays; the values
  // outside the tile are zeroed when stored
  auto load = [&](int kt) {
    const int64_t r0 = rb + (int64_t)kt * kSwTK + 8 * wave;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t r = r0 + e < re ? r0 + e : rb;
#pragma unroll
      for (int q = 0; q < NQ; ++q) rh[q][e] = H[r * c + (uvalid[q] ? c0 + ucls[q] : 0)];
      rw[e] = wsrc[omega ? r : 0];
    }
    const int64_t r = rb + (int64_t)kt * kSwTK + xr;
    rx = *reinterpret_cast<const f32x4*>(X + (r < re ? r : rb) * d + (xvalid ? xcol : 0));
  };
  auto store = [&](int buf, int kt) {
    const int64_t r0 = rb + (int64_t)kt * kSwTK + 8 * wave;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      float u[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float h = rh[q][e];
        u[e] = r0 + e < re && uvalid[q] ? (float)rw[e] * h * (1.f - h) : 0.f;
      }
      if constexpr (BF3) {
        bf16x8 hi, lo;
        split8(u, hi, lo);
        *reinterpret_cast<bf16x8*>(&Us[0][buf][ucls[q]][8 * wave]) = hi;
        *reinterpret_cast<bf16x8*>(&Us[1][buf][ucls[q]][8 * wave]) = lo;
      } else {
        *reinterpret_cast<f32x4*>(&Us[0][buf][ucls[q]][8 * wave]) = f32x4{u[0], u[1], u[2], u[3]};
        *reinterpret_cast<f32x4*>(&Us[0][buf][ucls[q]][8 * wave + 4]) =
            f32x4{u[4], u[5], u[6], u[7]};
      }
    }
    const int64_t r = rb + (int64_t)kt * kSwTK + xr;
    const bool ok = r < re && xvalid;
    float* dst = xp < 4 ? &XaT[buf][4 * xp][xr] : &XbT[buf][4 * (xp - 4)][xr];
#pragma unroll
    for (int e = 0; e < 4; ++e) dst[e * kSwXS] = ok ? rx[e] : 0.f;
  };

  const int64_t nrows = re > rb ? re - rb : 0;
  const int nk = (int)((nrows + kSwTK - 1) / kSwTK);
  if (nk > 0) {
    load(0);
    store(0, 0);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    load(kt + 1);   // past the last stage every row is out of range (stored as zero, never read)
    __builtin_amdgcn_sched_barrier(0);
    // this lane's pairs: (a0 + 4 wave + j, b0 + li).  The u of class block i + 1 is read while
    // block i's MFMAs run (the scheduler is kept from hoisting all of them, which would not fit
    // two waves per SIMD)
    if constexpr (BF3) {
      const f32x4 xb0 = *reinterpret_cast<const f32x4*>(&XbT[buf][li][8 * g]);
      const f32x4 xb1 = *reinterpret_cast<const f32x4*>(&XbT[buf][li][8 * g + 4]);
      bf16x8 bh[4], bl[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 xa0 = *reinterpret_cast<const f32x4*>(&XaT[buf][4 * wave + j][8 * g]);
        const f32x4 xa1 = *reinterpret_cast<const f32x4*>(&XaT[buf][4 * wave + j][8 * g + 4]);
        const float pr[8] = {xa0[0] * xb0[0], xa0[1] * xb0[1], xa0[2] * xb0[2], xa0[3] * xb0[3],
                             xa1[0] * xb1[0], xa1[1] * xb1[1], xa1[2] * xb1[2], xa1[3] * xb1[3]};
        split8(pr, bh[j], bl[j]);
      }
      bf16x8 ah = *reinterpret_cast<const bf16x8*>(&Us[0][buf][li][8 * g]);
      bf16x8 al = *reinterpret_cast<const bf16x8*>(&Us[1][buf][li][8 * g]);
#pragma unroll
      for (int i = 0; i < CMW; ++i) {
        const int in = i + 1 < CMW ? i + 1 : i;
        const bf16x8 nh = *reinterpret_cast<const bf16x8*>(&Us[0][buf][16 * in + li][8 * g]);
        const bf16x8 nl = *reinterpret_cast<const bf16x8*>(&Us[1][buf][16 * in + li][8 * g]);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma3(ah, al, bh[j], bl[j], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        ah = nh;
        al = nl;
      }
    } else {
#pragma unroll
      for (int kg = 0; kg < kSwTK / 16; ++kg) {
        const int k0 = 16 * kg + 4 * g;
        const f32x4 xb = *reinterpret_cast<const f32x4*>(&XbT[buf][li][k0]);
        f32x4 bv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 xa = *reinterpret_cast<const f32x4*>(&XaT[buf][4 * wave + j][k0]);
          bv[j] = f32x4{xa[0] * xb[0], xa[1] * xb[1], xa[2] * xb[2], xa[3] * xb[3]};
        }
        f32x4 av = *reinterpret_cast<const f32x4*>(&Us[0][buf][li][k0]);
#pragma unroll
        for (int i = 0; i < CMW; ++i) {
          const int in = i + 1 < CMW ? i + 1 : i;
          const f32x4 nv = *reinterpret_cast<const f32x4*>(&Us[0][buf][16 * in + li][k0]);
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], bv[j][q], acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          av = nv;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    store(buf ^ 1, kt + 1);
    __syncthreads();
  }

  float* out = part + (int64_t)sp * c * d * d;
  const int b = b0 + li;
#pragma unroll
  for (int i = 0; i < CMW; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a = a0 + 4 * wave + j;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = c0 + 16 * i + 4 * g + v;
        if (k < c && a < d && b < d && b <= a) out[((int64_t)k * d + a) * d + b] = acc[i][j][v];
      }
    }
}

// The Gram GEMM of contexts with FP32 arithmetic: tiles of 16 a x 16 b pairs against all classes
// of a class tile (up to 128), wave w taking a columns 4 w .. 4 w + 3 against all 16 b columns and
// CMW class blocks, so that a pair product x_a x_b is formed once per workgroup.  Both operands
// come packed (k_gram_pack): u = omega h (1 - h) and x, in stages of 32 rows of a split, as the
// 1 KB blocks of 16 rows x 16 columns that a wave reads from LDS as one 16-byte vector a lane,
// zero outside the split and past c and d.
// Beside FP32 MFMA a SIMD issues about one other vector instruction per MFMA, so what bounds the
// kernel is the MFMA rate as long as little else is issued: here four products per 4 CMW MFMAs
// and the copies.  Formed and bounds-checked in the kernel (once per pair tile, 136 times at
// d = 256), u and x took a third of the time: c = 100, d = 256, N = 200100 17.1 -> 11.8 ms (132
// TFLOP/s of 153), c = 200, d = 383, N = 60200 25.7 -> 15.2 ms, with the packing's 0.13 ms, CMW
// fitted to c (100 classes: 7 blocks, not 8) and the equal runs below (16.3 and 19.9 ms without).
// The order of the rows of an accumulator's sum is that of the kernels which read X and H as they
// are: instruction q of a 16-row block takes rows 4 g + q (kGramWide) or 4 q + g.
constexpr int kGramMaxWgs = 4092, kGramMinStages = 16, kGramCutStages = 16;
constexpr int64_t kGramFlagBytes = 16384;   // a flag a workgroup, the counter
template <bool WIDE>
__global__ __launch_bounds__(256) void k_gram_pack(const float* __restrict__ X,
                                                   const float* __restrict__ H,
                                                   const double* __restrict__ omega, int64_t N,
                                                   int d, int c, int64_t rps, int stage0, int T,
                                                   int nct, int cmw, int nab,
                                                   f32x4* __restrict__ U, f32x4* __restrict__ XP,
                                                   int32_t* __restrict__ done) {
  const int sp = blockIdx.x / T, t = blockIdx.x % T;
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int e = threadIdx.x; e <= kGramMaxWgs; e += 256) done[e] = 0;   // flags and counter
  const int64_t rb = (int64_t)sp * rps, re = rb + rps < N ? rb + rps : N;
  const int64_t r0 = rb + (int64_t)(stage0 + t) * 32;
  if (r0 >= re) return;   // never read
  const int nu = nct * cmw;
  f32x4* u = U + (int64_t)blockIdx.x * nu * 128;
  f32x4* xp = XP + (int64_t)blockIdx.x * nab * 128;
  for (int e = blockIdx.y * 512 + threadIdx.x, i = 0; i < 2; ++i, e += 256) {
    if (e >= (nu + nab) * 128) return;
    const int li = e & 15, g = (e >> 4) & 3, blk = e >> 6;
    const bool is_u = blk < 2 * nu;
    const int kg = is_u ? (blk / cmw) & 1 : (blk - 2 * nu) / nab;
    const int cb = is_u ? blk / (2 * cmw) * cmw + blk % cmw : (blk - 2 * nu) % nab;
    const int col = 16 * cb + li;
    f32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t r = r0 + 16 * kg + (WIDE ? 4 * g + q : 4 * q + g);
      float y = 0.f;
      if (is_u) {
        if (r < re && col < c) {
          const float h = H[r * c + col];
          y = (omega ? (float)omega[r] : 1.f) * h * (1.f - h);
        }
      } else if (r < re && col < d) {
        y = X[r * d + col];
      }
      v[q] = y;
    }
    if (is_u) u[e] = v;
    else xp[e - nu * 128] = v;
  }
}

// Stages [stage0, stage0 + nkc) of every unit (class tile, pair tile, split); later ranges go on
// from the sums in `part`.  With more units than workgroups the stages of all units, end to end,
// are cut into equal runs, one a workgroup (units alone leave the last round of workgroups nearly
// empty: 1088 units on 512 slots at d = 256, c = 100).  A run is at least a unit long, so a unit
// is cut at most once, and its sum is carried over the cut through `part`: a workgroup takes the
// head of its last unit first and the tail of its first unit last, for which the workgroup before
// it has then had as much time as the head takes.  Runs are dealt by a counter in the order in which
// workgroups start, so the workgroup waited for is running, whatever else the device runs and in
// whatever order its dies take workgroups, and its head waits for nothing: the wait ends.
// Ranges of under 16 stages (the rest that the scratch left over) are not cut.  From there on the
// preconditioner with and without cuts: c = 200, d = 383 2.41 -> 2.38 ms at 16 stages, 2.85 -> 2.64 at
// 47, 7.5 -> 5.3 at 375; c = 100, d = 256 1.15 -> 1.07 ms at 20 stages, 1.39 -> 1.23 at 32; with many
// units a workgroup they cost what they gain (c = 300, d = 400: 5.24 -> 5.27 ms at 17 stages, 7.28 ->
// 7.18 at 157).
// workgroups that a CU's registers hold
constexpr int gram_wgs_per_cu(int cmw) {
  return cmw <= 1 ? 7 : cmw <= 2 ? 5 : cmw <= 3 ? 4 : cmw <= 5 ? 3 : 2;
}
template <int CMW>
__global__ __launch_bounds__(256, gram_wgs_per_cu(CMW)) void k_gram(
    const f32x4* __restrict__ U, const f32x4* __restrict__ XP, int64_t N, int d, int c,
    const int32_t* __restrict__ tiles, int ntiles, int units, int nct, int nab, int64_t rps,
    int stage0, int nkc, int T, float* part, int32_t* done) {
  constexpr int NB = 2 * (CMW + 2), NL = (NB + 3) / 4;   // 1 KB blocks of a stage, per wave
  __shared__ f32x4 sm[2][NB * 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int li = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ int ticket;
  int id = blockIdx.x;
  if ((int)gridDim.x < units) {   // units may be cut
    if (tid == 0) ticket = atomicAdd(done + kGramMaxWgs, 1);
    __syncthreads();
    id = __builtin_amdgcn_readfirstlane(ticket);
  }
  const int64_t total = (int64_t)units * nkc, run = (total + gridDim.x - 1) / gridDim.x;
  const int64_t lo = id * run, hi = lo + run < total ? lo + run : total;
  if (lo >= hi) return;
  const int u0 = (int)(lo / nkc), u1 = (int)((hi - 1) / nkc);

  for (int n = 0; n <= u1 - u0; ++n) {
    // the last unit first, then the whole ones, then the first
    const int u = n == 0 ? u1 : n == u1 - u0 ? u0 : u0 + n;
    const int kb = u == u0 ? (int)(lo - (int64_t)u * nkc) : 0;
    const int ke = u == u1 ? (int)(hi - (int64_t)u * nkc) : nkc;
    const int cls_t = u % nct, pt = u / nct % ntiles, sp = u / nct / ntiles;
    const int A = tiles[2 * pt], B = tiles[2 * pt + 1];
    const int c0 = cls_t * 16 * CMW, a0 = 16 * A, b0 = 16 * B;
    const int64_t rb = (int64_t)sp * rps;
    const int64_t nrows = (rb + rps < N ? rb + rps : N) - rb;
    const int all = nrows > 0 ? (int)((nrows + 31) / 32) - stage0 : 0;   // the split's stages
    const int kn = ke < all ? ke : all;
    const bool resume = stage0 > 0 || kb > 0;
    float* out = part + (int64_t)sp * c * d * d;
    const int b = b0 + li;
    if (kb > 0) {
      if (tid == 0)
        while (__hip_atomic_load(done + id - 1, __ATOMIC_ACQUIRE,
                                 __HIP_MEMORY_SCOPE_AGENT) == 0)
          __builtin_amdgcn_s_sleep(8);
      __syncthreads();
    }

    f32x4 acc[CMW][4];
#pragma unroll
    for (int i = 0; i < CMW; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (resume) {
          const int a = a0 + 4 * wave + j;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int k = c0 + 16 * i + 4 * g + v;
            if (k < c && a < d && b <= a) acc[i][j][v] = out[((int64_t)k * d + a) * d + b];
          }
        }
      }

    // block m of a stage: CMW of u per 16 rows, then a's and b's
    const f32x4* src[NL];
    int step[NL];
#pragma unroll
    for (int m = 0; m < NL; ++m) {
      const int blk = wave + 4 * m, x = blk - 2 * CMW;   // x: a, a, b, b
      if (x < 0) {
        src[m] = U + ((((int64_t)sp * T + kb) * nct + cls_t) * 2 * CMW + blk) * 64 + lane;
        step[m] = nct * 2 * CMW * 64;
      } else {
        src[m] = XP + (((int64_t)sp * T + kb) * 2 * nab + (x & 1) * nab + (x < 2 ? A : B)) * 64 +
                 lane;
        step[m] = 2 * nab * 64;
      }
    }
    f32x4 st[NL];
    auto load = [&]() {
#pragma unroll
      for (int m = 0; m < NL; ++m)
        if (wave + 4 * m < NB) {
          st[m] = *src[m];
          src[m] += step[m];
        }
    };
    auto store = [&](int buf) {
#pragma unroll
      for (int m = 0; m < NL; ++m)
        if (wave + 4 * m < NB) sm[buf][(wave + 4 * m) * 64 + lane] = st[m];
    };
    if (kb < kn) {
      load();
      store(kb & 1);
    }
    __syncthreads();
    for (int kt = kb; kt < kn; ++kt) {
      const int buf = kt & 1;
      if (kt + 1 < kn) load();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kg = 0; kg < 2; ++kg) {
        const f32x4* us = &sm[buf][kg * CMW * 64 + lane];
        const f32x4 xb = sm[buf][(2 * CMW + 2 + kg) * 64 + lane];
        f32x4 bv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 xa = sm[buf][(2 * CMW + kg) * 64 + 16 * g + 4 * wave + j];
          bv[j] = f32x4{xa[0] * xb[0], xa[1] * xb[1], xa[2] * xb[2], xa[3] * xb[3]};
        }
        f32x4 av = us[0];
#pragma unroll
        for (int i = 0; i < CMW; ++i) {
          const f32x4 nv = us[(i + 1 < CMW ? i + 1 : i) * 64];
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], bv[j][q], acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          av = nv;
        }
      }
      if (kt + 1 < kn) store(buf ^ 1);
      __syncthreads();
    }

#pragma unroll
    for (int i = 0; i < CMW; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int a = a0 + 4 * wave + j;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = c0 + 16 * i + 4 * g + v;
          if (k < c && a < d && b <= a) out[((int64_t)k * d + a) * d + b] = acc[i][j][v];
        }
      }
    if (ke < nkc) {
      // Every wave waits for its own stores before the barrier (which does not wait for them: a barrier
      // orders within the workgroup), so that all the sums are in L2 when thread 0 writes L2 back and
      // sets the flag; a release by every thread would write L2 back 256 times (235 us, so 126).
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0)
        __hip_atomic_store(done + id, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// P[k][a][b] = sum over splits (in order, FP64) of the lower-triangle entry (max, min) +
// shift [a == b]: P is exactly symmetric.
template <typename T>
__global__ __launch_bounds__(256) void k_syrk_reduce(const T* __restrict__ part, int S, int c,
                                                     int d, double shift,
                                                     double* __restrict__ P) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t dd = (int64_t)d * d;
  if (idx >= (int64_t)c * dd) return;
  const int64_t k = idx / dd;
  const int rem = (int)(idx - k * dd);
  const int a = rem / d, b = rem - (rem / d) * d;
  const int64_t e = k * dd + (a >= b ? (int64_t)a * d + b : (int64_t)b * d + a);
  double acc = 0.0;
  for (int p = 0; p < S; ++p) acc += (double)part[(int64_t)p * c * dd + e];
  P[idx] = acc + (a == b ? shift : 0.0);
}

// In-place right-looking Cholesky of block k (lower triangle); upper part zeroed.
// A non-positive (or NaN) pivot records k in *bad (smallest k wins) and stops the block.
__global__ __launch_bounds__(256) void k_chol(double* __restrict__ P, int d, int32_t* bad) {
  const int k = blockIdx.x;
  double* A = P + (int64_t)k * d * d;
  const int tid = threadIdx.x;
  for (int j = 0; j < d; ++j) {
    __syncthreads();
    const double piv = A[(int64_t)j * d + j];
    if (!(piv > 0.0)) {
      if (tid == 0) atomicMin(bad, k);
      return;
    }
    const double ljj = sqrt(piv);
    const double inv = 1.0 / ljj;
    __syncthreads();
    if (tid == 0) A[(int64_t)j * d + j] = ljj;
    for (int i = j + 1 + tid; i < d; i += blockDim.x) A[(int64_t)i * d + j] *= inv;
    __syncthreads();
    const int m = d - j - 1;
    for (int e = tid; e < m * m; e += blockDim.x) {
      const int ii = e / m, kk = e % m;
      if (kk <= ii) {
        const int i = j + 1 + ii, q = j + 1 + kk;
        A[(int64_t)i * d + q] -= A[(int64_t)i * d + j] * A[(int64_t)q * d + j];
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < d * d; e += blockDim.x) {
    const int i = e / d, q = e % d;
    if (q > i) A[e] = 0.0;
  }
}

// Pinv_k = (L_k L_k^T)^-1, one column per thread: forward solve L y = e_j, then L^T x = y.
// All lanes walk the same (i, p) sequence (entries above the unit's row are zero), so the
// factor reads are uniform across the wave and the column reads/writes are coalesced.
__global__ __launch_bounds__(256) void k_chol_inv(const double* __restrict__ L,
                                                  double* __restrict__ Pinv, int d,
                                                  const int32_t* bad) {
  if (*bad != INT_MAX) return;
  const int k = blockIdx.x;
  const double* Lk = L + (int64_t)k * d * d;
  double* Y = Pinv + (int64_t)k * d * d;
  for (int j0 = 0; j0 < d; j0 += blockDim.x) {
    const int j = j0 + threadIdx.x;
    const bool on = j < d;
    for (int i = 0; i < d; ++i) {
      double acc = (i == j) ? 1.0 : 0.0;
      for (int p = 0; p < i; ++p) acc -= Lk[(int64_t)i * d + p] * (on ? Y[(int64_t)p * d + j] : 0.0);
      if (on) Y[(int64_t)i * d + j] = acc / Lk[(int64_t)i * d + i];
    }
    for (int i = d - 1; i >= 0; --i) {
      double acc = on ? Y[(int64_t)i * d + j] : 0.0;
      for (int p = i + 1; p < d; ++p) acc -= Lk[(int64_t)p * d + i] * (on ? Y[(int64_t)p * d + j] : 0.0);
      if (on) Y[(int64_t)i * d + j] = acc / Lk[(int64_t)i * d + i];
    }
  }
}

// Cholesky factor and inverse of block k in one pass, the whole block held in registers.
// The symmetric sweep operator on pivot j maps a -> a - a_{:j} a_{j:} / a_jj off row/column j,
// a_{j:} / a_jj on them and -1/a_jj on the pivot; sweeping every pivot of an SPD matrix leaves
// -P^-1.  Before pivot j is swept its unswept column is the Schur complement, so
// L[i][j] = a_ij / sqrt(a_jj) (i >= j) is the Cholesky factor, and a_jj <= 0 means P is not SPD.
// Thread (ty, tx) of a TT x TT grid owns rows ty + TT u and columns tx + TT v (u, v < TB).
// L is written over P (P is read completely before the first pivot).
template <int TT, int TB>
__global__ __launch_bounds__(TT* TT) void k_sweep(double* __restrict__ P, double* __restrict__ Pinv,
                                                  int d, int32_t* bad, int write_l) {
  const int kb = blockIdx.x;
  double* A0 = P + (int64_t)kb * d * d;
  double* Y = Pinv + (int64_t)kb * d * d;
  const int ty = threadIdx.x / TT, tx = threadIdx.x % TT;
  __shared__ double prow[TT * TB];
  double a[TB][TB];
#pragma unroll
  for (int u = 0; u < TB; ++u)
#pragma unroll
    for (int v = 0; v < TB; ++v) {
      const int i = ty + TT * u, q = tx + TT * v;
      a[u][v] = (i < d && q < d) ? A0[(int64_t)i * d + q] : 0.0;
    }
  __syncthreads();
  for (int j = 0; j < d; ++j) {
    const int uj = j / TT;
    if (ty == j % TT) {
#pragma unroll
      for (int u = 0; u < TB; ++u)
        if (u == uj) {
#pragma unroll
          for (int v = 0; v < TB; ++v) prow[tx + TT * v] = a[u][v];
        }
    }
    __syncthreads();
    const double piv = prow[j];
    if (!(piv > 0.0)) {
      if (threadIdx.x == 0) atomicMin(bad, kb);
      return;
    }
    const double ip = 1.0 / piv;
    // the factor's column j (only when asked: each step's barrier then waits for these stores)
    if (write_l && tx == 0) {
      const double sq = sqrt(piv);
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        const int i = ty + TT * u;
        if (i >= j && i < d) A0[(int64_t)i * d + j] = i == j ? sq : prow[i] / sq;
      }
    }
    // rank-1 update of every element, then row j, column j and the pivot rewritten (their
    // owners are known: j = jt + TT vj in both the row and the column decomposition)
    double pri[TB], pc[TB];
#pragma unroll
    for (int u = 0; u < TB; ++u) pri[u] = prow[ty + TT * u] * ip;
#pragma unroll
    for (int v = 0; v < TB; ++v) pc[v] = prow[tx + TT * v];
#pragma unroll
    for (int u = 0; u < TB; ++u)
#pragma unroll
      for (int v = 0; v < TB; ++v) a[u][v] = fma(-pri[u], pc[v], a[u][v]);
    const int jt = j % TT, vj = j / TT;
#pragma unroll
    for (int u = 0; u < TB; ++u)
      if (u == vj && ty == jt) {
#pragma unroll
        for (int v = 0; v < TB; ++v) a[u][v] = pc[v] * ip;       // row j: a_jq / a_jj
      }
#pragma unroll
    for (int v = 0; v < TB; ++v)
      if (v == vj && tx == jt) {
#pragma unroll
        for (int u = 0; u < TB; ++u) a[u][v] = pri[u];           // column j: a_ij / a_jj
#pragma unroll
        for (int u = 0; u < TB; ++u)
          if (u == vj && ty == jt) a[u][v] = -ip;                // pivot
      }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < TB; ++u)
#pragma unroll
    for (int v = 0; v < TB; ++v) {
      const int i = ty + TT * u, q = tx + TT * v;
      if (i < d && q < d) {
        Y[(int64_t)i * d + q] = -a[u][v];
        if (write_l && q > i) A0[(int64_t)i * d + q] = 0.0;
      }
    }
}

constexpr int kSwLD = 17;   // row stride of a 16 x 16 block in LDS (odd: no bank conflicts by column)

// x of one lane, uniform
__device__ __forceinline__ double lane_value(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// the value of lane P of each row of 16 lanes
template <int P> __device__ __forceinline__ double row_lane(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x150 + P, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x150 + P, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sweep of the 16 x 16 pivot block in `Kb` (row stride kSwLD), in place, by one wave: lane (q, r) =
// (l / 16, l % 16) holds row r, columns 4 q + k.  KIND names the form whose products and roundings it
// takes (each form has its own).  Co[p][r]: what a column's sweep needs of pivot p, T_p[r]
// (kSweepRows) or column p (kSweepPanel); Ro[p]: row p before its sweep; Ip[p]: 1 / pivot.  False when
// a pivot is not positive.  What bounds it: the chain from pivot to pivot (update, 1 / pivot, product,
// update); row p comes to the other rows by a broadcast within 16 lanes and column p by a permute,
// both beside the division.
enum SweepKind { kSweepRows, kSweepPanel, kSweepBlock };
template <int KIND, int P>
__device__ __forceinline__ bool sweep16_step(double (&b)[4], double* Co, double* Ro, double* Ip,
                                             int r, int q, int lane) {
  const double piv = lane_value(b[P & 3], P + 16 * (P >> 2));
  const double ip = 1.0 / piv;
  double apc[4];   // M[P][4 q + k]
#pragma unroll
  for (int k = 0; k < 4; ++k) apc[k] = row_lane<P>(b[k]);
  double x;        // kSweepRows: M[P][r], else M[r][P]
  if (KIND == kSweepRows) {
    double y[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] = __shfl(apc[k], 16 * (r >> 2), 64);
    x = (r & 2) ? ((r & 1) ? y[3] : y[2]) : ((r & 1) ? y[1] : y[0]);
  } else {
    x = __shfl(b[P & 3], r + 16 * (P >> 2), 64);
  }
  const double pri = x * ip;
  if (KIND != kSweepBlock) {
    if (q == 0) Co[P * 16 + r] = KIND == kSweepRows ? pri : x;
    if (r == P) {
#pragma unroll
      for (int k = 0; k < 4; ++k) Ro[P * 16 + 4 * q + k] = b[k];
    }
    if (lane == 0) Ip[P] = ip;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = 4 * q + k;
    const double u = KIND != kSweepPanel ? fma(-pri, apc[k], b[k]) : fma(-(x * apc[k]), ip, b[k]);
    b[k] = r != P ? (c != P ? u : pri) : (c != P ? apc[k] * ip : -ip);
  }
  return piv > 0.0;
}
template <int KIND, int... P>
__device__ __forceinline__ bool sweep16_steps(double (&b)[4], double* Co, double* Ro, double* Ip,
                                              int lane, std::integer_sequence<int, P...>) {
  bool ok = true;
  ((ok = sweep16_step<KIND, P>(b, Co, Ro, Ip, lane & 15, lane >> 4, lane) && ok), ...);
  return ok;
}
template <int KIND>
__device__ __forceinline__ bool sweep16(double* Kb, double* Co, double* Ro, double* Ip, int lane) {
  const int r = lane & 15, cg = (lane >> 4) * 4;
  double b[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) b[k] = Kb[r * kSwLD + cg + k];
  const bool ok =
      sweep16_steps<KIND>(b, Co, Ro, Ip, lane, std::make_integer_sequence<int, 16>{});
#pragma unroll
  for (int k = 0; k < 4; ++k) Kb[r * kSwLD + cg + k] = b[k];
  return ok;
}

// Inverse of each SPD block (d <= 128) by the sweep operator taken sixteen pivots at a time,
// for callers that do not ask for the factor.  Sweeping a pivot block K of the current
// (symmetric) M gives M_KK <- N = -M_KK^-1, M_IK <- T_I = -M_IK N (and M_KI <- T_I^T),
// M_IJ <- M_IJ - T_I M_KJ for the other rows and columns, the same matrix as sweeping K's
// pivots one at a time; after every block M = -P^-1.  M's 16 x 16 tiles stay in registers (padding:
// identity), the diagonal ones in wave 0, the others dealt to seven waves.  Per block K: the column
// panel is in LDS and N known; -T by FP64 MFMA, one tile a wave; then every wave updates its tiles by
// MFMA and writes the next panel, while wave 0 updates the next pivot block first and sweeps it: two
// barriers a block.  The products and sums are those of the form without MFMA (256 threads, the
// pivot block between barriers), in its order (an FP64 MFMA adds its products one by one): solves in
// FP32 keep their bits.  What bounds it: the chain of the pivots (sweep16; with its rows through LDS
// 46 us).  c = 10, d = 100: 49 -> 38 us; c = 50, d = 50: 20.5 -> 16.6 us.
template <int D16>
__global__ __launch_bounds__(512) void k_sweep_blk(const double* __restrict__ P,
                                                   double* __restrict__ Pinv, int d,
                                                   int32_t* bad) {
  constexpr int DP = 16 * D16, LD = kSwLD, NOFF = D16 * (D16 - 1), NT = D16 > NOFF / 7 ? D16 : (NOFF + 6) / 7;
  __shared__ double PK[2][DP * LD];   // [i][m] column panel M[i][K0 + m], two in turn
  __shared__ double Ts[DP * LD];      // [i][m] -T
  __shared__ double Kb[2][16 * LD];   // N, two in turn
  __shared__ int fail;
  const int kb = blockIdx.x, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, g = lane >> 4;
  const double* A0 = P + (int64_t)kb * d * d;
  // tile n of this wave (in the MFMA's result layout: rows g + 4 v of column li)
  auto tile_of = [&](int n, int& I, int& J) {
    if (wave == 0) {
      I = J = n;
      return n < D16;
    }
    const int e = wave - 1 + 7 * n, i = e / (D16 > 1 ? D16 - 1 : 1), j = e - i * (D16 - 1);
    I = i;
    J = j + (j >= i);
    return e < NOFF;
  };
  f64x4 t[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    int I, J;
    const bool on = tile_of(n, I, J);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * I + g + 4 * v, j = 16 * J + li;
      t[n][v] = on && i < d && j < d ? A0[(int64_t)i * d + j] : (i == j ? 1.0 : 0.0);
    }
  }
  // the tile's part of panel K
  auto dump = [&](int K) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      int I, J;
      if (!tile_of(n, I, J) || J != K) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) PK[K & 1][(16 * I + g + 4 * v) * LD + li] = t[n][v];
    }
  };
  auto pivots = [&](const f64x4& x, int K) {   // by wave 0
    double* kbk = Kb[K & 1];
#pragma unroll
    for (int v = 0; v < 4; ++v) kbk[(g + 4 * v) * LD + li] = x[v];
    wave_lds_fence();
    if (!sweep16<kSweepBlock>(kbk, nullptr, nullptr, nullptr, lane) && lane == 0) {
      fail = 1;
      atomicMin(bad, kb);
    }
  };
  if (threadIdx.x == 0) fail = 0;
  if (wave == 0) {
    wave_lds_fence();
    pivots(t[0], 0);
  }
  dump(0);
  __syncthreads();
#pragma unroll
  for (int K = 0; K < D16; ++K) {
    if (fail) return;   // the same for every thread
    const double* pk = PK[K & 1];
    const double* nk = Kb[K & 1];
    // -T[i][c] = sum_m M[i][K0 + m] N[m][c]
    if (wave < D16) {
      f64x4 u = Mfma16<double>::zero();
#pragma unroll
      for (int q = 0; q < 4; ++q)
        u = __builtin_amdgcn_mfma_f64_16x16x4f64(pk[(16 * wave + li) * LD + 4 * q + g],
                                                 nk[(4 * q + g) * LD + li], u, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) Ts[(16 * wave + g + 4 * v) * LD + li] = u[v];
    }
    __syncthreads();
    auto update = [&](f64x4& x, int I, int J) {
      if (I != K && J != K) {   // M_IJ -= T_I M_KJ (M_KJ[m][j] = M[j][K0 + m] by symmetry)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          x = __builtin_amdgcn_mfma_f64_16x16x4f64(Ts[(16 * I + li) * LD + 4 * q + g],
                                                   pk[(16 * J + li) * LD + 4 * q + g], x, 0, 0, 0);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          x[v] = I == J ? nk[(g + 4 * v) * LD + li]
                        : J == K ? -Ts[(16 * I + g + 4 * v) * LD + li]
                                 : -Ts[(16 * J + li) * LD + g + 4 * v];
      }
    };
    if (wave == 0 && K + 1 < D16) {
      update(t[K + 1], K + 1, K + 1);
      pivots(t[K + 1], K + 1);
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      int I, J;
      if (tile_of(n, I, J) && !(wave == 0 && n == K + 1)) update(t[n], I, J);
    }
    if (K + 1 < D16) dump(K + 1);
    __syncthreads();
  }
  double* Y = Pinv + (int64_t)kb * d * d;
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    int I, J;
    const bool on = tile_of(n, I, J);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * I + g + 4 * v, j = 16 * J + li;
      if (on && i < d && j < d) Y[(int64_t)i * d + j] = -t[n][v];
    }
  }
}

// Inverse of each SPD block of 128 < d <= 576 for callers that do not ask for the factor: the
// sweeps above and below, sixteen pivots at a time and with the update of the other rows on FP64
// MFMA, bit for bit: every element takes the same products and sums, rounded in the same order
// (an FP64 MFMA adds its four products one after the other, each with one rounding).  A solve in
// FP32 rounds M^-1 r, and what flips there moves its result by far more than the inverse's own
// error, so the inverse keeps its bits.
// ROWS (d <= 256, as k_sweep): row p before its sweep is R_p, T_p = R_p / pivot, and every other
// row takes M[r][q] -= T_p[r] R_p[q], p by p; column p becomes T_p.  Else (as k_sweep_glb): the
// rows of the panel are swept as a whole, and the others take M[i][j] -= sum_m Bo[m][i] Rs[m][j]
// with Bo the rows as loaded and Rs as swept; columns of the panel are Rs transposed.
// Per panel of sixteen rows: thread q takes column q of the panel into registers and sweeps it with
// the coefficients of each pivot (in LDS), no barrier between pivots; the two operand panels go to
// LDS and the waves update 16 x 16 tiles in place in the output (they do not fit a CU's registers
// and LDS at d = 256), kInvTiles at a time from a common counter, while wave 0 first updates the
// next pivot block and sweeps it for its coefficients.
// What bounds it: the tiles' passes through one CU's path to L2, then the FP64 rate.
// 100 blocks of 256: 4.08 ms with one pivot and two barriers of 1024 threads at a time (k_sweep)
// -> 0.41 ms; 200 blocks of 383: 8.75 ms with the panels and tiles of k_sweep_glb -> 1.8 ms.
constexpr int kInvMaxD = 576, kInvTiles = 4;
// row pitch of the LDS panels: 16 mod 32 doubles, so that the two k of half a wave's read meet no
// bank twice
template <bool ROWS> constexpr int kInvPitch = ROWS ? 272 : 592;

template <bool ROWS>
__global__ __launch_bounds__(1024) void k_inv_mfma(const double* P, double* Pinv, int d,
                                                   int32_t* bad) {
  const int kb = blockIdx.x, lane = threadIdx.x & 63, tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, g = lane >> 4;
  constexpr int dp = kInvPitch<ROWS>;
  const int nb = (d + 15) / 16;
  __shared__ double Lp[16 * dp];   // [16][dp] the left operand: -T or Bo
  __shared__ double Rp[16 * dp];   // [16][dp] the right operand: R or Rs
  __shared__ double Kb[16 * kSwLD];
  __shared__ __align__(16) double Co[256], Ro[256], Ip[16];
  __shared__ int fail, next;
  const double* A0 = P + (int64_t)kb * d * d;
  double* Y = Pinv + (int64_t)kb * d * d;

  // element (row, col) of the block as it stands; outside it the identity
  auto load = [&](const double* src, int I, int J) {
    f64x4 t;
    const int col = 16 * J + li;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int row = 16 * I + g + 4 * w;
      t[w] = row < d && col < d ? src[(int64_t)row * d + col] : (row == col ? 1.0 : 0.0);
    }
    return t;
  };
  auto update = [&](const f64x4& t, int I, int J) {
    f64x4 c = ROWS ? t : Mfma16<double>::zero();
#pragma unroll
    for (int k = 0; k < 4; ++k)
      c = __builtin_amdgcn_mfma_f64_16x16x4f64(Lp[(4 * k + g) * dp + 16 * I + li],
                                               Rp[(4 * k + g) * dp + 16 * J + li], c, 0, 0, 0);
    return ROWS ? c : t - c;
  };
  auto pivots = [&](const f64x4& t) {   // by wave 0
#pragma unroll
    for (int w = 0; w < 4; ++w) Kb[(g + 4 * w) * kSwLD + li] = t[w];
    wave_lds_fence();
    if (!sweep16<ROWS ? kSweepRows : kSweepPanel>(Kb, Co, Ro, Ip, lane) && lane == 0) {
      fail = 1;
      atomicMin(bad, kb);
    }
  };

  if (wave == 0) {
    if (lane == 0) fail = 0;
    pivots(load(A0, 0, 0));
  }
  __syncthreads();
  if (fail) return;   // the same for every thread
  for (int K = 0; K < nb; ++K) {
    const double* src = K == 0 ? A0 : Y;
    const int k0 = 16 * K, q = tid;
    const bool last = K + 1 == nb;
    if (tid == 0) next = 0;
    if (q < 16 * nb) {
      double v[16];
      if (q >= k0 && q < k0 + 16) {
        // of R_p, tile column q takes what follows its own pivot (its start is T_q, below)
#pragma unroll
        for (int p = 0; p < 16; ++p) {
          v[p] = Kb[p * kSwLD + q - k0];
          Rp[p * dp + q] = ROWS ? (p > q - k0 ? Ro[p * 16 + q - k0] : 0.0) : v[p];
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          v[r] = k0 + r < d && q < d ? src[(int64_t)(k0 + r) * d + q] : 0.0;
        if (!ROWS) {
#pragma unroll
          for (int p = 0; p < 16; ++p) Lp[p * dp + q] = v[p];
        }
#pragma unroll
        for (int p = 0; p < 16; ++p) {
          const double R = v[p], ip = Ip[p], T = R * ip;
          if (ROWS) {
            Rp[p * dp + q] = R;
            Lp[p * dp + q] = -T;
          }
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (r != p) {
              const double c = Co[p * 16 + r];
              v[r] = ROWS ? fma(-c, R, v[r]) : fma(-(c * R), ip, v[r]);
            }
          v[p] = T;
        }
        if (!ROWS) {
#pragma unroll
          for (int p = 0; p < 16; ++p) Rp[p * dp + q] = v[p];
        }
      }
      if (q < d) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (k0 + r < d) Y[(int64_t)(k0 + r) * d + q] = last ? -v[r] : v[r];
      }
    }
    __syncthreads();
    if (wave == 0 && !last) pivots(update(load(src, K + 1, K + 1), K + 1, K + 1));
    // tiles (I, J) with I != K, numbered row by row; the next pivot block goes no further
    const int nt = (nb - 1) * nb;
    for (;;) {
      int id0 = 0;
      if (lane == 0) id0 = atomicAdd(&next, kInvTiles);
      id0 = __builtin_amdgcn_readfirstlane(id0);
      if (id0 >= nt) break;
      f64x4 t[kInvTiles];
      int I[kInvTiles], J[kInvTiles];
      const int i0 = (int)((unsigned)id0 / (unsigned)nb), j0 = id0 - i0 * nb;
#pragma unroll
      for (int n = 0; n < kInvTiles; ++n) {
        const int wrap = j0 + n >= nb, i = i0 + wrap;   // nb >= 9 > kInvTiles: at most one row on
        I[n] = i + (i >= K);
        J[n] = j0 + n - (wrap ? nb : 0);
        if (I[n] >= nb) I[n] = J[n] = -1;
        if (I[n] < 0) continue;
        if (J[n] != K) {
          t[n] = load(src, I[n], J[n]);
        } else {
#pragma unroll
          for (int w = 0; w < 4; ++w) {   // T_q of the tile's rows; else Rs transposed
            const int at = li * dp + 16 * I[n] + g + 4 * w;
            t[n][w] = ROWS ? -Lp[at] : Rp[at];
          }
        }
      }
#pragma unroll
      for (int n = 0; n < kInvTiles; ++n) {
        if (I[n] < 0 || (I[n] == K + 1 && J[n] == K + 1)) continue;
        const f64x4 x = ROWS || J[n] != K ? update(t[n], I[n], J[n]) : t[n];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int row = 16 * I[n] + g + 4 * w, col = 16 * J[n] + li;
          if (row < d && col < d) Y[(int64_t)row * d + col] = last ? -x[w] : x[w];
        }
      }
    }
    __syncthreads();   // the tiles, the LDS panels and the next pivot block
    if (fail) return;  // the same for every thread
  }
}

typedef void (*InvKernel)(const double*, double*, int, int32_t*);
// d <= 128 has the form with its tiles in registers (k_sweep_blk); past d = 576 the two panels leave
// LDS.  Between, the MFMA form was the faster one at every size measured, k_sweep or k_sweep_glb ->
// it: two blocks of 129 0.157 -> 0.121 ms, of 160 0.193 -> 0.146, of 256 3.86 -> 0.41, of 257 2.89
// -> 0.49, of 576 23.0 -> 3.8; 300 blocks of 129 0.329 -> 0.269, of 256 8.6 -> 1.04, of 384 18.4 ->
// 4.0, of 576 56 -> 14.
static InvKernel pick_inv(int d) {
  if (d <= 128 || d > kInvMaxD) return nullptr;
  return d <= 256 ? k_inv_mfma<true> : k_inv_mfma<false>;
}
// The sweep for blocks too large for registers (d > 256): block kb is copied to Pinv and swept
// there in global memory, NB pivots at a time.  With the block partitioned at pivots K as
// [[K, B^T], [B, D]], sweeping K leaves [[-K^-1, K^-1 B^T], [B K^-1, D - B K^-1 B^T]].  The NB
// rows of K are staged in LDS twice: as loaded (Bo = [K, B^T], whose columns outside K are B^T)
// and swept pivot by pivot (Rs, ending as [-K^-1, K^-1 B^T]); then every row outside K is updated
// from LDS, D[i][j] -= sum_m Bo[m][i] Rs[m][j] and A[i][k] = Rs[k][i] for k in K (the block stays
// symmetric), four rows by four columns per thread, and the rows of K are written from Rs.
// Before pivot p is swept, its staged row holds column p of the Schur complement, so the
// Cholesky factor's column p is that row over sqrt(pivot) (written to P when asked).  After all
// pivots the block holds -P^-1.  LDS: ((2 NB + 1) d + NB) doubles (NB = 16: 99 KB at d = 384;
// NB = 8 for larger blocks, at twice the passes over the block).
template <int NB>
__global__ __launch_bounds__(256) void k_sweep_glb(double* __restrict__ P, double* __restrict__ Pinv,
                                                   int d, int32_t* bad, int write_l) {
  extern __shared__ __align__(16) double sw_lds[];
  double* Bo = sw_lds;                  // [NB][d] rows of K as loaded
  double* Rs = sw_lds + NB * d;         // [NB][d] rows of K as swept
  double* Rm = sw_lds + 2 * NB * d;     // [d] pivot row before its sweep
  double* Cp = Rm + d;                  // [NB] pivot column before its sweep
  const int kb = blockIdx.x, tid = threadIdx.x;
  double* L = P + (int64_t)kb * d * d;
  double* A = Pinv + (int64_t)kb * d * d;
  for (int64_t e = tid; e < (int64_t)d * d; e += 256) A[e] = L[e];
  __syncthreads();
  const int nq = (d + 3) / 4;            // 4 x 4 tiles of the block
  for (int k0 = 0; k0 < d; k0 += NB) {
    const int nb = d - k0 < NB ? d - k0 : NB;
    for (int e = tid; e < nb * d; e += 256) {
      const int m = e / d, j = e - m * d;
      const double v = A[(int64_t)(k0 + m) * d + j];
      Bo[m * d + j] = v;
      Rs[m * d + j] = v;
    }
    __syncthreads();
    for (int m = 0; m < nb; ++m) {
      const int pc = k0 + m;
      const double piv = Rs[m * d + pc];
      if (!(piv > 0.0)) {
        if (tid == 0) atomicMin(bad, kb);
        return;
      }
      const double ip = 1.0 / piv;
      const double rs = write_l ? 1.0 / sqrt(piv) : 0.0;
      // the pivot row and column as they stand, so that every staged element can then be
      // updated in place by the one thread that owns it
      for (int j = tid; j < d; j += 256) {
        const double v = Rs[m * d + j];
        Rm[j] = v;
        if (write_l && j >= pc) L[(int64_t)j * d + pc] = v * rs;   // factor column pc
      }
      if (tid < nb) Cp[tid] = Rs[tid * d + pc];
      __syncthreads();
      for (int e = tid; e < nb * d; e += 256) {
        const int r = e / d, j = e - r * d;
        double v;
        if (r == m) v = j == pc ? -ip : Rm[j] * ip;
        else if (j == pc) v = Cp[r] * ip;
        else v = Rs[e] - Cp[r] * Rm[j] * ip;
        Rs[e] = v;
      }
      __syncthreads();
    }
    // rows outside K: D -= B K^-1 B^T, and the columns of K from Rs; 4 x 4 tiles
    for (int t = tid; t < nq * nq; t += 256) {
      const int i0 = 4 * (t / nq), j0 = 4 * (t % nq);
      double acc[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v] = 0.0;
      for (int m = 0; m < nb; ++m) {
        double bi[4], rj[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          bi[u] = i0 + u < d ? Bo[m * d + i0 + u] : 0.0;
          rj[u] = j0 + u < d ? Rs[m * d + j0 + u] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[u][v] = fma(bi[u], rj[v], acc[u][v]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u;
        if (i >= d) continue;
        const bool iin = i >= k0 && i < k0 + nb;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int j = j0 + v;
          if (j >= d) continue;
          const bool jin = j >= k0 && j < k0 + nb;
          double* a = A + (int64_t)i * d + j;
          if (iin) *a = Rs[(i - k0) * d + j];
          else if (jin) *a = Rs[(j - k0) * d + i];
          else *a -= acc[u][v];
        }
      }
    }
    __syncthreads();
  }
  for (int64_t e = tid; e < (int64_t)d * d; e += 256) {
    A[e] = -A[e];
    if (write_l) {
      const int i = (int)(e / d), j = (int)(e - (int64_t)i * d);
      if (j > i) L[e] = 0.0;
    }
  }
}

typedef void (*SweepBlkKernel)(const double*, double*, int, int32_t*);

static SweepBlkKernel pick_sweep_blk(int d) {
  if (d > 128) return nullptr;
  switch ((d + 15) / 16) {
    case 1: return k_sweep_blk<1>;
    case 2: return k_sweep_blk<2>;
    case 3: return k_sweep_blk<3>;
    case 4: return k_sweep_blk<4>;
    case 5: return k_sweep_blk<5>;
    case 6: return k_sweep_blk<6>;
    case 7: return k_sweep_blk<7>;
    default: return k_sweep_blk<8>;
  }
}

typedef void (*SweepKernel)(double*, double*, int, int32_t*, int);

static SweepKernel pick_sweep(int d, int* threads) {
  if (d <= 128) {
    *threads = 256;
    switch ((d + 15) / 16) {
      case 1: return k_sweep<16, 1>;
      case 2: return k_sweep<16, 2>;
      case 3: return k_sweep<16, 3>;
      case 4: return k_sweep<16, 4>;
      case 5: return k_sweep<16, 5>;
      case 6: return k_sweep<16, 6>;
      case 7: return k_sweep<16, 7>;
      default: return k_sweep<16, 8>;
    }
  }
  if (d <= 256) {
    *threads = 1024;
    switch ((d + 31) / 32) {
      case 5: return k_sweep<32, 5>;
      case 6: return k_sweep<32, 6>;
      case 7: return k_sweep<32, 7>;
      default: return k_sweep<32, 8>;
    }
  }
  return nullptr;
}

__global__ void k_bad_reset(Status* st) { st->bad_block = INT_MAX; }

// Tile shape by c: class blocks per wave (CMW) and waves along the classes (WC); pair tiles
// of 16 x BR with BR = PNW (4 / WC), PNW = 4 (FP32) or 2 (FP64).  The bf16x3 kernel: CMW = 8,
// WC = 1 (its four waves along the pairs), pair tiles of 16 x 16.
struct SyrkShape {
  int cmw, wc, pnw;
  int tc() const { return 16 * cmw * wc; }
  int br() const { return pnw * (4 / wc); }
};
int gram_form_for(int prec, int d, int c, const void* X) {
  if (prec == FIRAL_F64 || c <= 64 || d % 4 != 0 || ((uintptr_t)X & 15) != 0) return kGramClassic;
  const char* w = getenv("FIRAL_GRAM_WIDE");
  if (w && atoi(w) == 0) return kGramClassic;
  const char* g3 = getenv("FIRAL_BF3_GRAM");
  return prec == FIRAL_BF16X3 && g3 && atoi(g3) != 0 ? kGramWideBf3 : kGramWide;
}
SyrkShape syrk_shape(int prec, int c, int form) {
  if (form != kGramClassic) return SyrkShape{8, 1, 4};
  const int pnw = prec == FIRAL_F64 ? 2 : 4;
  if (c <= 16) return SyrkShape{1, 1, pnw};
  if (c <= 32) return SyrkShape{1, 2, pnw};
  if (c <= 64) return SyrkShape{2, 2, pnw};
  return SyrkShape{4, 2, pnw};
}

// Blocks of 256 < d <= kSweepGlbMaxD go to the global-memory sweep: 16-pivot panels up to
// d = 600, 8-pivot panels up to 1200 (its LDS, ((2 NB + 1) d + NB) doubles, fits the 160 KB of
// a CU up to there); larger ones to the column-at-a-time factor and inverse.
constexpr int kSweepGlb16MaxD = 600, kSweepGlbMaxD = 1200;
template <int NB>
constexpr int sweep_glb_lds(int d) { return ((2 * NB + 1) * d + NB) * (int)sizeof(double); }
static DeviceOnce g_sweep_glb_attr;

static int sweep_glb_launch(double* P, double* Pinv, int d, int c, int32_t* bad, bool want_l,
                            hipStream_t st) {
  if (!g_sweep_glb_attr.done()) {
    FIRAL_HIP(hipFuncSetAttribute((const void*)k_sweep_glb<16>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  sweep_glb_lds<16>(kSweepGlb16MaxD)));
    FIRAL_HIP(hipFuncSetAttribute((const void*)k_sweep_glb<8>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  sweep_glb_lds<8>(kSweepGlbMaxD)));
    g_sweep_glb_attr.set();
  }
  if (d <= kSweepGlb16MaxD)
    k_sweep_glb<16><<<c, 256, sweep_glb_lds<16>(d), st>>>(P, Pinv, d, bad, want_l ? 1 : 0);
  else
    k_sweep_glb<8><<<c, 256, sweep_glb_lds<8>(d), st>>>(P, Pinv, d, bad, want_l ? 1 : 0);
  FIRAL_LAUNCHED();
  return FIRAL_OK;
}

template <typename T, int CMW, int WC>
static void launch_syrk(Ctx* x, const double* omega, int64_t rps, hipStream_t st) {
  constexpr int PNW = sizeof(T) == 4 ? 4 : 2;
  const int nct = (int)cdiv(x->c, 16 * CMW * WC);
  const int64_t nwg = (int64_t)nct * x->syrk_ntiles * x->syrk_splits;
  k_syrk<T, T, CMW, PNW, WC><<<(unsigned)nwg, 256, 0, st>>>(
      (const T*)x->X, (const T*)x->H, omega, x->N, x->d, x->c, x->syrk_tiles, x->syrk_ntiles, nct,
      rps, (T*)x->syrk_part);
}

// Class tiles and blocks of k_gram: as few tiles of at most 128 classes, cut alike.
static void gram_shape(int c, int* nct, int* cmw) {
  *nct = (int)cdiv(c, 128);
  *cmw = (int)cdiv(cdiv(c, *nct), 16);
}
// Bytes of one stage of every split, packed.
static int64_t gram_stage_bytes(const Ctx* x) {
  int nct, cmw;
  gram_shape(x->c, &nct, &cmw);
  return (int64_t)x->syrk_splits * (nct * cmw + cdiv(x->d, 16)) * 2048;
}
// Scratch that a context holds at least (its product buffer, mostly larger): 32 stages a split, so
// that taking the sums out of `part` and back is little beside them, or all there are.
int64_t gram_min_bytes(const Ctx* x) {
  return kGramFlagBytes +
         gram_stage_bytes(x) * std::min<int64_t>(32, cdiv(cdiv(x->N, x->syrk_splits), 32));
}

static int gram_launch(Ctx* x, const double* omega, int64_t rps, hipStream_t st) {
  int nct, cmw;
  gram_shape(x->c, &nct, &cmw);
  const int nab = (int)cdiv(x->d, 16), S = x->syrk_splits;
  const int64_t stages = cdiv(rps, 32);
  const int T = (int)std::min<int64_t>(
      stages, ((int64_t)x->g_bytes - kGramFlagBytes) / gram_stage_bytes(x));
  int32_t* done = (int32_t*)x->G;
  f32x4* U = (f32x4*)((char*)x->G + kGramFlagBytes);
  f32x4* XP = U + (int64_t)S * T * nct * cmw * 128;
  auto pack = x->gram_form == kGramClassic ? k_gram_pack<false> : k_gram_pack<true>;
  typedef void (*K)(const f32x4*, const f32x4*, int64_t, int, int, const int32_t*, int, int, int,
                    int, int64_t, int, int, int, float*, int32_t*);
  static const K kernels[8] = {k_gram<1>, k_gram<2>, k_gram<3>, k_gram<4>,
                               k_gram<5>, k_gram<6>, k_gram<7>, k_gram<8>};
  const int units = nct * x->syrk_ntiles * S;
  for (int64_t s0 = 0; s0 < stages; s0 += T) {
    const int nkc = (int)std::min<int64_t>(T, stages - s0);
    const int wgs = nkc < kGramCutStages
                        ? units : std::min({units, x->n_cu * gram_wgs_per_cu(cmw), kGramMaxWgs});
    pack<<<dim3((unsigned)(S * T), (unsigned)cdiv(nct * cmw + nab, 4)), 256, 0, st>>>((const float*)x->X, (const float*)x->H, omega, x->N,
                                            x->d, x->c, rps, (int)s0, T, nct, cmw, nab, U, XP,
                                            done);
    FIRAL_LAUNCHED();
    kernels[cmw - 1]<<<(unsigned)wgs, 256, 0, st>>>(U, XP, x->N, x->d, x->c, x->syrk_tiles,
                                                    x->syrk_ntiles, units, nct, nab, rps, (int)s0,
                                                    nkc, T, (float*)x->syrk_part, done);
    FIRAL_LAUNCHED();
  }
  return FIRAL_OK;
}

template <typename T>
static int precond_t(Ctx* x, const double* omega, double shift, bool want_l, hipStream_t st) {
  const int d = x->d, c = x->c;
  const int S = x->syrk_splits;
  const int64_t rps = cdiv(x->N, S);
  k_bad_reset<<<1, 1, 0, st>>>(x->status);
  FIRAL_LAUNCHED();
  const SyrkShape sh = syrk_shape(x->prec, c, x->gram_form);
  if (x->gram_packed) {
    FIRAL_CHECK(gram_launch(x, omega, rps, st));
  } else if (x->gram_form != kGramClassic) {
    const int nct = (int)cdiv(c, sh.tc());
    const int64_t nwg = (int64_t)nct * x->syrk_ntiles * S;
    auto k = x->gram_form == kGramWideBf3 ? k_syrkw<8, true> : k_syrkw<8, false>;
    k<<<(unsigned)nwg, 256, 0, st>>>((const float*)x->X, (const float*)x->H, omega, x->N, d, c,
                                     x->syrk_tiles, x->syrk_ntiles, nct, rps,
                                     (float*)x->syrk_part);
  } else if (sh.wc == 1) launch_syrk<T, 1, 1>(x, omega, rps, st);
  else if (sh.cmw == 1) launch_syrk<T, 1, 2>(x, omega, rps, st);
  else if (sh.cmw == 2) launch_syrk<T, 2, 2>(x, omega, rps, st);
  else launch_syrk<T, 4, 2>(x, omega, rps, st);
  FIRAL_LAUNCHED();
  const int64_t n = (int64_t)c * d * d;
  k_syrk_reduce<T><<<(unsigned)cdiv(n, 256), 256, 0, st>>>((const T*)x->syrk_part, S, c, d,
                                                           shift, x->P);
  FIRAL_LAUNCHED();
  int threads = 0;
  SweepKernel sw = pick_sweep(d, &threads);
  SweepBlkKernel sb = want_l ? nullptr : pick_sweep_blk(d);
  InvKernel iv = want_l ? nullptr : pick_inv(d);
  if (sb) {
    sb<<<c, 512, 0, st>>>(x->P, x->Pinv, d, &x->status->bad_block);
    FIRAL_LAUNCHED();
  } else if (iv) {
    iv<<<c, 1024, 0, st>>>(x->P, x->Pinv, d, &x->status->bad_block);
    FIRAL_LAUNCHED();
  } else if (sw) {
    sw<<<c, threads, 0, st>>>(x->P, x->Pinv, d, &x->status->bad_block, want_l ? 1 : 0);
    FIRAL_LAUNCHED();
  } else if (d <= kSweepGlbMaxD) {
    FIRAL_CHECK(sweep_glb_launch(x->P, x->Pinv, d, c, &x->status->bad_block, want_l, st));
  } else {
    k_chol<<<c, 256, 0, st>>>(x->P, d, &x->status->bad_block);
    FIRAL_LAUNCHED();
    k_chol_inv<<<c, 256, 0, st>>>(x->P, x->Pinv, d, &x->status->bad_block);
    FIRAL_LAUNCHED();
  }
  return FIRAL_OK;
}

// Pair tiles (a-block of 16, b-block of BR) that meet the lower triangle, and the row-split
// count, for a context (host side, at creation).  Grids smaller than the device's workgroup
// slots (two per CU) are split over the rows up to about 1024 workgroups (partials within
// 256 MB); larger grids of the wide forms take the split count (up to 8, partials within 4 GiB)
// with the least time in rounds of slots, ceil(wgs S / slots) / S: at configuration 4, 2400
// workgroups on 512 slots run 4.69 rounds unsplit (five, the last one two-thirds empty) and
// 18.75 in four splits (nineteen quarter-length rounds).
void syrk_plan(int prec, int d, int c, int form, int n_cu, std::vector<int32_t>* tiles,
               int* splits) {
  const SyrkShape sh = syrk_shape(prec, c, form);
  const int BR = sh.br();
  const int nab = (int)cdiv(d, 16), nbb = (int)cdiv(d, BR);
  tiles->clear();
  for (int A = 0; A < nab; ++A)
    for (int Bb = 0; Bb < nbb && Bb * BR <= 16 * A + 15; ++Bb) {
      tiles->push_back(A);
      tiles->push_back(Bb);
    }
  const int64_t nt = (int64_t)tiles->size() / 2;
  const int64_t wgs = nt * cdiv(c, sh.tc());
  const int64_t es = prec == FIRAL_F64 ? 8 : 4;
  const int64_t blk = (int64_t)c * d * d * es;
  const int64_t slots = 2 * (int64_t)std::max(1, n_cu);
  if (form != kGramClassic && wgs >= slots) {
    const int64_t cap = std::min<int64_t>(8, std::max<int64_t>(1, ((int64_t)4 << 30) / blk));
    int S = 1;
    for (int64_t t = 2; t <= cap; ++t)   // rounds / S, compared as cross products
      if (cdiv(wgs * t, slots) * S < cdiv(wgs * S, slots) * t) S = (int)t;
    *splits = S;
    return;
  }
  const int64_t mem_cap = std::max<int64_t>(1, ((int64_t)1 << 28) / blk);
  *splits = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(cdiv(1024, wgs), 64),
                                                        mem_cap));
}

// Whether a context's Gram blocks are formed from packed operands, its pair tiles then 16 x 16: with
// FP32 arithmetic from sixteen stages of 32 rows a split on.  Below, the packing's launch costs what
// it saves or more (with the reduction): N = 300, d = 20, c = 5 (one stage) 0.030 -> 0.040 ms, N =
// 3000, d = 256, c = 100 (12 stages) 0.481 -> 0.487; from there on N = 20000, d = 100, c = 10 (17
// stages) 0.094 -> 0.083, N = 60000, d = 383, c = 70 13.3 -> 6.9.
bool gram_packed(const Ctx* x, std::vector<int32_t>* tiles) {
  if (x->prec == FIRAL_F64 || x->gram_form == kGramWideBf3 ||
      cdiv(cdiv(x->N, x->syrk_splits), 32) < kGramMinStages)
    return false;
  tiles->clear();
  for (int A = 0; 16 * A < x->d; ++A)
    for (int B = 0; B <= A; ++B) {
      tiles->push_back(A);
      tiles->push_back(B);
    }
  return true;
}

int chol_blocks_launch(double* P, double* Pinv, int d, int c, int32_t* bad, bool want_inv,
                       bool want_l, hipStream_t st) {
  int threads = 0;
  SweepKernel sw = pick_sweep(d, &threads);
  SweepBlkKernel sb = want_l ? nullptr : pick_sweep_blk(d);
  InvKernel iv = want_l ? nullptr : pick_inv(d);
  if (sb) {
    sb<<<c, 512, 0, st>>>(P, Pinv, d, bad);
    FIRAL_LAUNCHED();
  } else if (iv) {
    iv<<<c, 1024, 0, st>>>(P, Pinv, d, bad);
    FIRAL_LAUNCHED();
  } else if (sw) {
    sw<<<c, threads, 0, st>>>(P, Pinv, d, bad, want_l ? 1 : 0);
    FIRAL_LAUNCHED();
  } else if (d <= kSweepGlbMaxD) {
    FIRAL_CHECK(sweep_glb_launch(P, Pinv, d, c, bad, want_l, st));
  } else {
    k_chol<<<c, 256, 0, st>>>(P, d, bad);
    FIRAL_LAUNCHED();
    if (want_inv) {
      k_chol_inv<<<c, 256, 0, st>>>(P, Pinv, d, bad);
      FIRAL_LAUNCHED();
    }
  }
  return FIRAL_OK;
}

template <typename L, int CMW, int WC>
static void launch_gram64(const L* X, const L* H, const double* omega, int64_t N, int d, int c,
                          const int32_t* tiles, int ntiles, int S, double* part,
                          hipStream_t st) {
  const int nct = (int)cdiv(c, 16 * CMW * WC);
  const int64_t nwg = (int64_t)nct * ntiles * S;
  k_syrk<double, L, CMW, 2, WC><<<(unsigned)nwg, 256, 0, st>>>(X, H, omega, N, d, c, tiles, ntiles,
                                                               nct, cdiv(std::max<int64_t>(N, 1), S),
                                                               part);
}

template <typename L>
static int gram64_t(const L* X, const L* H, const double* omega, int64_t N, int d, int c,
                    const int32_t* tiles, int ntiles, int S, double shift, double* part,
                    double* out, hipStream_t st) {
  const SyrkShape sh = syrk_shape(FIRAL_F64, c, kGramClassic);
  if (sh.wc == 1) launch_gram64<L, 1, 1>(X, H, omega, N, d, c, tiles, ntiles, S, part, st);
  else if (sh.cmw == 1) launch_gram64<L, 1, 2>(X, H, omega, N, d, c, tiles, ntiles, S, part, st);
  else if (sh.cmw == 2) launch_gram64<L, 2, 2>(X, H, omega, N, d, c, tiles, ntiles, S, part, st);
  else launch_gram64<L, 4, 2>(X, H, omega, N, d, c, tiles, ntiles, S, part, st);
  FIRAL_LAUNCHED();
  const int64_t n = (int64_t)c * d * d;
  k_syrk_reduce<double><<<(unsigned)cdiv(n, 256), 256, 0, st>>>(part, S, c, d, shift, out);
  FIRAL_LAUNCHED();
  return FIRAL_OK;
}

int gram64_launch(int prec, const void* X, const void* H, const double* omega, int64_t N, int d,
                  int c, const int32_t* tiles, int ntiles, int S, double shift, double* part,
                  double* out, hipStream_t st) {
  if (prec == FIRAL_F64)
    return gram64_t<double>((const double*)X, (const double*)H, omega, N, d, c, tiles, ntiles, S,
                            shift, part, out, st);
  return gram64_t<float>((const float*)X, (const float*)H, omega, N, d, c, tiles, ntiles, S,
                         shift, part, out, st);
}

int precond_launch(Ctx* x, const double* omega, double shift, hipStream_t st, bool want_l) {
  if (x->prec == FIRAL_F64) return precond_t<double>(x, omega, shift, want_l, st);
  return precond_t<float>(x, omega, shift, want_l, st);
}

}  // namespace firal
