// Hessian product of Lemma 1 and the per-point gradient of eq. 11 on packed operands, for FP32 and
// bf16x3 contexts that the fused kernels (hvp_fused.hip) do not cover: d > 128, or more classes
// than a fused tile holds.
//
// Per chunk of R rows (columns n: the s c columns of the probe block, in tiles of 128):
//   k_pk_xv     G = X V on 128 x 128 tiles; its epilogue also sums, per row, G h over the columns
//               of each probe inside the tile
//   k_pk_alpha  alpha[p][r] = sum of those partial sums (FP64, fixed order)
//   k_pk_xtg    part[sp] (+)= X^T G' over the split's rows, G' = omega (G - alpha) h (the row step
//               of Lemma 1) formed while G is staged
// and the split sums are reduced in a fixed order (hvp.hip).  The gradient runs k_pk_xv on W, then
// on U with an epilogue that sums U^T x (G - alpha) h over the tile's columns.
//
// Arithmetic of the products (PkArith):
//   kPkF32  FP32 contexts: FP32 MFMA 16x16x4.
//   kPkB2   bf16x3 contexts: operands as two bf16 planes x_0 + x_1 (rounded to nearest even),
//           x_0 y_0 + x_0 y_1 + x_1 y_0 on the 16x16x32 bf16 MFMA, FP32 accumulation.
//
// Two forms of the row step (kept apart so that each problem keeps its order of summation):
//   flat     column tiles run over the s c columns without regard to probes; G is stored as it is,
//            the sums are FP64 (of FP32-rounded products up to c = 128), G' = omega ((G - alpha) h)
//   windows  (d > 128, c > 128, d a multiple of 4, of 8 in bf16x3) each probe's columns are cut into
//            windows of 128; E = omega G is stored, the window's sums of E h are FP32, their sum
//            over the windows (beta = omega alpha) FP64, G' = (E - beta) h
//
// Operand layout.  A block of 16 values of the free index by 32 of the contraction index k is two
// contiguous 1 KB halves in the order in which the MFMA takes it: lane (g, li) = 16 g + li holds 16
// bytes of free index li in each half, so every move of a block, from memory to registers or to LDS
// and back, is a contiguous 1 KB access without bank conflicts, and with the operands padded by
// zeros to whole blocks the main loops need no masks.
//   FP32 contexts  half h: k = 16 h + 4 q + g (flat) or 16 h + 4 g + q (windows), q = 0..3; one
//                  MFMA 16x16x4 per q
//   bf16x3         half p: plane p, k = 8 g + u, u = 0..7
//   X    [row block][k block]                 (context creation)
//   X^T  [32-row block][a block]              (context creation)
//   V    [column tile][k block][8 column blocks] (once per call)
//   G    [column tile][16-row block][8 column blocks] of 16 x 16 FP32 in the MFMA's result layout:
//        lane (g, li) holds result rows 4 g .. 4 g + 3 of column li
// The rows of each 32-row group are taken in the order (pk_row) that makes the lane's values of two
// G blocks exactly its eight k of the second contraction, so G' goes from G to the operand without
// leaving its lane.  Every per-row array of this file (H^T, alpha, omega) is in that order.  Packed
// rows start anew, on whole tiles, with each row chunk.
#include <algorithm>

#include <hip/hip_ext.h>

#include "common.h"

namespace firal {

namespace {

constexpr int kPkT = 128;             // rows and columns of a first-contraction tile
constexpr int kPkMaxWaves = 8;        // waves of a second-contraction workgroup

enum PkArith { kPkF32 = 0, kPkB2 = 1 };
enum PkMode { kPkFlat = 0, kPkWin = 1, kPkDot = 2, kPkFlatX = 3 };

typedef float f4 __attribute__((ext_vector_type(4)));

// Workgroup b of n runs on XCD b % 8; give each XCD a contiguous range of logical tiles.
__device__ __forceinline__ unsigned pk_lid(unsigned b, unsigned n) {
  const unsigned q = n >> 3, r = n & 7, x = b & 7, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

// Row (within its group of 32) at position pos: FP32 flat 16 b + 4 v + g, FP32 windows the
// position itself, bf16x3 8 g + 4 b + v, for pos = 16 b + 4 g + v.
enum PkOrder { kPkRowQ = 0, kPkRowId = 1, kPkRow8 = 2 };
template <int AR, bool WIN> constexpr int pk_order() {
  return AR == kPkB2 ? kPkRow8 : WIN ? kPkRowId : kPkRowQ;
}
__host__ __device__ __forceinline__ int pk_row(int order, int pos) {
  const int b = pos >> 4, g = (pos >> 2) & 3, v = pos & 3;
  return order == kPkRowQ ? 16 * b + 4 * v + g : order == kPkRowId ? pos : 8 * g + 4 * b + v;
}
// k (within its 32) of half h, element q of lane group g in FP32 contexts.
__device__ __forceinline__ int pk_k32(int order, int h, int g, int q) {
  return 16 * h + (order == kPkRowQ ? 4 * q + g : 4 * g + q);
}

// Eight FP32 values of a lane (two f4 in k order) as the two parts of an operand block.
template <int AR>
__device__ __forceinline__ void pk_parts_of(const f4 (&y)[2], f4 (&o)[2]) {
  if constexpr (AR == kPkF32) {
    o[0] = y[0];
    o[1] = y[1];
  } else {
    const float v[8] = {y[0][0], y[0][1], y[0][2], y[0][3], y[1][0], y[1][1], y[1][2], y[1][3]};
    bf16x8 hi, lo;
    split8(v, hi, lo);
    o[0] = __builtin_bit_cast(f4, hi);
    o[1] = __builtin_bit_cast(f4, lo);
  }
}

// An operand's values with those of rows at or beyond lim cleared (row(u): row of value u): eight
// bf16 or four FP32.
template <bool BF, typename F>
__device__ __forceinline__ f4 pk_keep(f4 x, int lim, F row) {
  if constexpr (BF) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const unsigned m =
          (row(2 * w) < lim ? 0xFFFFu : 0u) | (row(2 * w + 1) < lim ? 0xFFFF0000u : 0u);
      x[w] = __builtin_bit_cast(float, __builtin_bit_cast(unsigned, (float)x[w]) & m);
    }
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = row(v) < lim ? x[v] : 0.f;
  }
  return x;
}

// A unit of a stage: the wave's MI row blocks (a, registers) times two column blocks (b, registers).
// Every accumulator takes its products in the order of k (bf16: x_0 y_0, x_0 y_1, x_1 y_0); the 2 MI
// accumulators take turns.
template <int AR, int MI>
__device__ __forceinline__ void pk_unit(const f4 (&a)[MI][2], const f4 (&b)[2][2], int j0,
                                        f32x4 (&acc)[MI][8]) {
  if constexpr (AR == kPkF32) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int i = 0; i < MI; ++i)
            acc[i][j0 + q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][h][e], b[q][h][e],
                                                                  acc[i][j0 + q], 0, 0, 0);
  } else {
    constexpr int pa[3] = {0, 0, 1}, pb[3] = {0, 1, 0};
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int i = 0; i < MI; ++i)
          acc[i][j0 + q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, a[i][pa[t]]), __builtin_bit_cast(bf16x8, b[q][pb[t]]),
              acc[i][j0 + q], 0, 0, 0);
  }
}

// The LDS stage buffers of both kernels: one is read, the next is complete, the third is written, so
// that a unit's operands are read from LDS a unit ahead, across the stage barrier too.
constexpr int kPkBufs = 3, kPkBuf = 8 * 2 * 256;   // floats of one

__device__ __forceinline__ void pk_read(f4 (&b)[2][2], const float* buf, int j0, int lane) {
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int p = 0; p < 2; ++p)
      b[q][p] = *reinterpret_cast<const f4*>(buf + ((j0 + q) * 2 + p) * 256 + lane * 4);
}

// Keeps the compiler's scheduler from moving instructions across this point: the next stage's
// loads are issued before the stage's MFMAs and consumed only after them.
__device__ __forceinline__ void pk_order_fence() { __builtin_amdgcn_sched_barrier(0); }

// Sum over the 16 lanes that share a lane group, in every lane of it (fixed order).
__device__ __forceinline__ double row16_sum(double v) {
  v = dpp_add<0xB1, 0xF, 0xF>(v);    // quad_perm [1,0,3,2]
  v = dpp_add<0x4E, 0xF, 0xF>(v);    // quad_perm [2,3,0,1]
  v = dpp_add<0x141, 0xF, 0xF>(v);   // row_half_mirror
  v = dpp_add<0x140, 0xF, 0xF>(v);   // row_mirror
  return v;
}
// One step of a sum over lanes that halves the lane's 2 N values: it keeps the half its bit `up`
// selects and adds its partner's values of that half (the partner, by CTRL, has the other bit).
template <int N, int CTRL>
__device__ __forceinline__ void half_step(double (&t)[8], bool up) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double keep = up ? t[N + i] : t[i], send = up ? t[i] : t[N + i];
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(send), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(send), CTRL, 0xF, 0xF, true);
    t[i] = keep + __hiloint2double(hi, lo);
  }
}
template <int CTRL>
__device__ __forceinline__ float dpp_add_f(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                           0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row16_sum_f(float v) {
  v = dpp_add_f<0xB1>(v);
  v = dpp_add_f<0x4E>(v);
  v = dpp_add_f<0x141>(v);
  return dpp_add_f<0x140>(v);
}

// Column tile ct: its first column and its width.  Windows: tile ct is window ct / s of probe
// ct % s (consecutive tiles share the window's classes).
struct PkCols {
  int c, s, SC, nw;   // nw: windows per probe, 0 = flat
  __host__ __device__ __forceinline__ int tiles() const {
    return nw ? s * nw : (SC + kPkT - 1) / kPkT;
  }
  __device__ __forceinline__ void tile(int ct, int& n0, int& width) const {
    if (nw) {
      const int w = (int)((unsigned)ct / (unsigned)s), p = ct - w * s, col0 = w * kPkT;
      n0 = p * c + col0;
      width = c - col0 < kPkT ? c - col0 : kPkT;
    } else {
      n0 = ct * kPkT;
      width = SC - n0 < kPkT ? SC - n0 : kPkT;
    }
  }
  // whether pairs of column blocks beyond the tiles' widths are a tenth of all or more
  __host__ bool part() const {
    const int last = nw ? c - (nw - 1) * kPkT : SC - (tiles() - 1) * kPkT, n = nw ? nw : tiles();
    return 10 * (4 - (last + 31) / 32) >= 4 * n;
  }
  // partial-sum slots: flat tile ct and its probe p share slot ct + p (a step to the next column
  // either stays in both or moves on in one of them); windows p nw + w
  __host__ __device__ __forceinline__ int64_t slots() const { return (int64_t)tiles() + s; }
};

constexpr int kPkSegLd = kPkT + 1;   // LDS row stride of the narrow-probe epilogue
constexpr int kPkSegC = 64;          // probes narrower than this are summed through LDS

template <int MODE>
constexpr size_t pk_xv_lds() {
  const size_t main_b = (size_t)kPkBufs * kPkBuf * 4;
  const size_t seg_b = MODE == kPkFlat ? (size_t)4 * 16 * kPkSegLd * 4 : 0;
  return main_b > seg_b ? main_b : seg_b;
}

// Kernel 1: tile of 128 rows x 128 columns, four waves of 32 rows each.  X blocks go straight from
// memory to the wave's registers (no other wave reads them), the tile's V blocks through kPkBufs LDS
// buffers shared by the four; the next stage's loads are in flight during the stage's MFMAs.
// What bounds it: in FP32 the MFMA rate (the rest is the fill of the pipeline and the epilogue, whose
// vector instructions issue one per MFMA beside another wave's FP32 MFMA); with bf16 planes the
// tile's way from L2 and LDS to the matrix cores and G's way to memory.  The products as wholes,
// before (row-tiled tiles, or transposed operands staged through LDS) and now: d = 256, c = 100, s =
// 32, N = 200,100 bf16x3 5.58 -> 2.55 ms; d = 203, c = 37, s = 7, N = 30,048 FP32 197 -> 150 us; d =
// 384, c = 1000, s = 16, N = 1,282,000 FP32 296 -> 281 ms; the gradient at d = 256, c = 100, s = 32 FP32
// 11.0 -> 6.15 ms.
// kPkDot: dpart[ct][row] = sum over the tile's columns of G_u (G - alpha) h, G and alpha those of
// the earlier kPkFlat call on W.
template <int AR, int MODE>
__global__ __launch_bounds__(256, 3) void k_pk_xv(
    const float* __restrict__ Xp, int nkb, int64_t R, const float* __restrict__ Vp, PkCols cols,
    const float* __restrict__ HT, int64_t ldh, const double* __restrict__ omega,
    float* __restrict__ G, int64_t nrb, double* __restrict__ apart, int64_t ldb,
    const float* __restrict__ alpha, double* __restrict__ dpart, Skip skip) {
  if (skip_now(skip)) return;
  extern __shared__ __align__(16) unsigned char pk_lds[];
  float* Bs = reinterpret_cast<float*>(pk_lds);   // [3][8][2][1 KB]
  constexpr int order = pk_order<AR, MODE == kPkWin>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, g = lane >> 4;
  const int nct = cols.tiles(), c = cols.c;
  // tiles in groups of 8 row tiles: consecutive logical ids take the 8 row tiles of a group for
  // one column tile, then the next column tile, so that the workgroups resident on one XCD share
  // 8 tiles of X and a few of V in its L2 (the last group may hold fewer row tiles)
  const unsigned lid = pk_lid(blockIdx.x, gridDim.x), nrt = (unsigned)((R + kPkT - 1) / kPkT);
  const unsigned grp = lid / (8u * nct), in = lid - grp * 8u * nct;
  const unsigned gsz = nrt - grp * 8 < 8 ? nrt - grp * 8 : 8;
  const int ct = (int)(gsz == 8 ? in >> 3 : in / gsz);
  const int64_t rt = grp * 8 + (in - (unsigned)ct * gsz);
  const int64_t row0 = rt * kPkT + 32 * wave;
  int n0, width;
  cols.tile(ct, n0, width);
  // pairs of column blocks within the tile's width (uniform); the others' products are zero
  const int units = (width + 31) >> 5;

  f32x4 acc[2][8];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // uniform bases: the lane's share of an address is a constant 32-bit offset
  const float* xw = Xp + (row0 >> 4) * nkb * 512;
  const float* vt = Vp + (int64_t)ct * nkb * kPkBuf;
  f4 bn[4], bu[2][2][2];
  auto load_a = [&](f4 (&r)[2][2], int kb) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        r[i][h] = reinterpret_cast<const f4*>(xw + ((int64_t)i * nkb + kb) * 512 + h * 256)[lane];
  };
  auto load_b = [&](int kb) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      bn[t] = reinterpret_cast<const f4*>(vt + (int64_t)kb * kPkBuf + t * 1024)[tid];
  };
  auto store_b = [&](int buf) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      *reinterpret_cast<f4*>(Bs + buf * kPkBuf + t * 1024 + tid * 4) = bn[t];
  };
  const int last = nkb - 1;
  // past the last stage the loads repeat it into buffers whose values are not used
  int rd = 0, nx = 1, wr = 2;
  // one stage with the operand a; the next stage's raw operand is loaded into r
  auto stage = [&](const f4 (&a)[2][2], f4 (&r)[2][2], int kb) {
    const float* b = Bs + rd * kPkBuf;
    load_a(r, kb < last ? kb + 1 : last);
    load_b(kb + 2 <= last ? kb + 2 : last);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u == 3) store_b(wr);
      if (u < 3)
        pk_read(bu[(u + 1) & 1], b, 2 * u + 2, lane);
      else
        pk_read(bu[0], Bs + nx * kPkBuf, 0, lane);
      pk_order_fence();
      if (u < units) pk_unit<AR, 2>(a, bu[u & 1], 2 * u, acc);
      pk_order_fence();
    }
    const int t = rd;
    rd = nx;
    nx = wr;
    wr = t;
    __syncthreads();
  };
  f4 r0[2][2], r1[2][2];   // the operands as loaded, two sets in turn
  load_a(r0, 0);
  load_b(0);
  store_b(0);
  load_b(last > 0 ? 1 : 0);
  store_b(1);
  __syncthreads();
  pk_read(bu[0], Bs, 0, lane);
  int kb = 0;
  for (; kb + 1 < nkb; kb += 2) {
    stage(r0, r1, kb);
    stage(r1, r0, kb + 1);
  }
  if (kb < nkb) stage(r0, r1, kb);

  // Epilogue.  Lane (g, li) of block (i, j) holds positions row0 + 16 i + 4 g + v, v = 0..3, of
  // column n0 + 16 j + li of the tile.  Columns beyond the tile's width have zero G.  Positions beyond the call's rows hold other rows' values or zero: the second kernel
  // clears them.  Every load is issued before the first is used.  VALU work here competes with the
  // other workgroup's MFMAs for issue, so the sums use as few operations as their order allows.
  float* gt = G + ((int64_t)ct * nrb + (row0 >> 4)) * 2048;   // uniform
  // probe and class of the tile's first column, and the last probe
  const int p_lo = (int)((unsigned)n0 / (unsigned)c), k_lo = n0 - p_lo * c;
  const int p_hi = (int)((unsigned)(n0 + width - 1) / (unsigned)c);
  f4 h[2][8];
  const float* hp[8];
  int pj[8];   // probe of the lane's column (kPkDot)
  {
    const float* h0 = HT + row0 + 4 * g;
    unsigned k = k_lo + li;   // class of the lane's column, counted on past the tile's width
    int p = p_lo;
    if (c < kPkSegC) {
      p += k / (unsigned)c;
      k %= (unsigned)c;
    } else {
      p += k >= (unsigned)c;
      k = min(k, k - c);   // k - c wraps to a large value below c
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      pj[j] = MODE == kPkDot ? min(p, cols.s - 1) : 0;
      hp[j] = reinterpret_cast<const float*>(reinterpret_cast<const char*>(h0) +
                                             (uint64_t)k * (unsigned)(4 * ldh));
      if constexpr (MODE != kPkDot) {
        h[0][j] = *reinterpret_cast<const f4*>(hp[j]);
        h[1][j] = *reinterpret_cast<const f4*>(hp[j] + 16);
      }
      k += 16;
      if (c < 16) {
        p += k / (unsigned)c;
        k %= (unsigned)c;
      } else {
        p += k >= (unsigned)c;
        k = min(k, k - c);
      }
    }
  }
  if constexpr (MODE == kPkDot) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float* ap = alpha + row0 + 16 * i + 4 * g;
      double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int j0 = 0; j0 < 8; j0 += 4) {   // four columns' loads at a time (registers)
        f4 e[4], al[4], hv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          e[q] = reinterpret_cast<const f4*>(gt + (i * 8 + j0 + q) * 256)[lane];
          hv[q] = *reinterpret_cast<const f4*>(hp[j0 + q] + 16 * i);
          al[q] = *reinterpret_cast<const f4*>(
              reinterpret_cast<const char*>(ap) + (uint64_t)(unsigned)pj[j0 + q] * (unsigned)(4 * ldb));
        }
        pk_order_fence();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (16 * (j0 + q) >= width) continue;   // uniform
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float x = acc[i][j0 + q][v] * ((e[q][v] - al[q][v]) * hv[q][v]);
            t[v] += (double)(16 * (j0 + q) + li < width ? x : 0.f);
          }
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) t[v] = row16_sum(t[v]);
      if (li == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t r = row0 + pk_row(order, 16 * i + 4 * g + v);
          if (r < R) dpart[(int64_t)ct * R + r] = t[v];
        }
      }
    }
    return;
  } else {
    if constexpr (MODE == kPkWin) {
      float om[2][4];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t r = row0 + pk_row(order, 16 * i + 4 * g + v);
          om[i][v] = omega ? (float)omega[r < R ? r : 0] : 1.f;
        }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] *= om[i][v];
    }
    // non-temporal: a chunk's G is read back by the second kernel from HBM, and should not evict X,
    // V and h from L2
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        __builtin_nontemporal_store(f4{acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]},
                                    reinterpret_cast<f4*>(gt + (i * 8 + j) * 256) + lane);
    if constexpr (MODE == kPkWin) {
      // FP32 sums over the window's two halves of 64 columns, then their sum
      const int w = ct / cols.s, p = ct - w * cols.s;
      double* ap = apart + ((int64_t)p * cols.nw + w) * ldb + row0 + 4 * g;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float t[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        if (width == kPkT) {
#pragma unroll
          for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              t[j >> 2][v] = fmaf(acc[i][j][v], h[i][j][v], t[j >> 2][v]);
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * j + li < width)
                t[j >> 2][v] = fmaf(acc[i][j][v], h[i][j][v], t[j >> 2][v]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) t[0][v] = row16_sum_f(t[0][v]) + row16_sum_f(t[1][v]);
        if (li == 0) {
#pragma unroll
          for (int v = 0; v < 4; ++v) ap[16 * i + v] = (double)t[0][v];
        }
      }
    } else if (c >= kPkSegC) {
      // at most three probes: each summed over the lane's columns, then over the 16 lanes.  FP32
      // products up to c = 128 (kPkFlat), exact ones beyond (kPkFlatX)
      if constexpr (MODE == kPkFlat) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] *= h[i][j][v];
      }
      auto term = [&](int i, int j, int v, float x) {
        if constexpr (MODE == kPkFlat) return (double)x;
        float y = h[i][j][v];
        asm("" : "+v"(x), "+v"(y));   // keeps the conversions inside the probe loop (registers)
        return (double)x * (double)y;
      };
      for (int p = p_lo; p <= p_hi; ++p) {
        const int lo = p * c - n0, hi = min(lo + c, width);   // its columns within the tile
        double t[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          // uniform branches: the block lies outside the probe, inside it, or is cut by its edge
          if (16 * j + 16 <= lo || 16 * j >= hi) continue;
          if (16 * j >= lo && 16 * j + 16 <= hi) {
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] += term(e >> 2, j, e & 3, acc[e >> 2][j][e & 3]);
          } else {
            const bool on = 16 * j + li >= lo && 16 * j + li < hi;
#pragma unroll
            for (int e = 0; e < 8; ++e)
              t[e] += term(e >> 2, j, e & 3, on ? acc[e >> 2][j][e & 3] : 0.f);
          }
        }
        // value e = 4 i + v ends in the lanes with li / 2 = e
        half_step<4, 0x140>(t, (li & 8) != 0);   // row_mirror
        half_step<2, 0x141>(t, (li & 4) != 0);   // row_half_mirror
        half_step<1, 0x1B>(t, (li & 2) != 0);    // quad_perm [3,2,1,0]
        const double sum = dpp_add<0xB1, 0xF, 0xF>(t[0]);
        if ((li & 1) == 0)
          apart[(int64_t)(ct + p) * ldb + row0 + 16 * (li >> 3) + 4 * g + ((li >> 1) & 3)] = sum;
      }
    } else if constexpr (MODE == kPkFlat) {
      // narrow probes: 16 x 128 products at a time through the wave's own LDS rows (the pipeline
      // buffers are free after the last barrier), one lane per (row, probe)
      float* seg = reinterpret_cast<float*>(pk_lds) + wave * 16 * kPkSegLd;
      for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            seg[(4 * g + v) * kPkSegLd + 16 * j + li] =
                i == 0 ? acc[0][j][v] * h[0][j][v] : acc[1][j][v] * h[1][j][v];
        __builtin_amdgcn_wave_barrier();
        for (int it = lane; it < 16 * (p_hi - p_lo + 1); it += 64) {
          const int rr = it & 15, p = p_lo + (it >> 4);
          const int lo = max(p * c - n0, 0), hi = min((p + 1) * c - n0, width);
          double t = 0.0;
          for (int m = lo; m < hi; ++m) t += (double)seg[rr * kPkSegLd + m];
          apart[(int64_t)(ct + p) * ldb + row0 + 16 * i + rr] = t;
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
}

// alpha[p][pos] (windows: beta = omega alpha) from the partial sums, for every position of the
// chunk's whole tiles; flat: also the row weights in position order (zero beyond the call's rows).
__global__ __launch_bounds__(256) void k_pk_alpha(const double* __restrict__ apart, PkCols cols,
                                                  int64_t Rp, int64_t ldb, int64_t R, int order,
                                                  const double* __restrict__ omega,
                                                  float* __restrict__ alpha,
                                                  float* __restrict__ omf, Skip skip) {
  if (skip_now(skip)) return;
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int p = blockIdx.y;
  if (pos >= Rp) return;
  double a = 0.0;
  if (cols.nw) {
    for (int w = 0; w < cols.nw; ++w) a += apart[((int64_t)p * cols.nw + w) * ldb + pos];
  } else {
    const int c = cols.c, ct1 = ((p + 1) * c - 1) / kPkT;
    for (int ct = p * c / kPkT; ct <= ct1; ++ct) a += apart[(int64_t)(ct + p) * ldb + pos];
    if (p == 0) {
      const int64_t r = (pos & ~(int64_t)31) + pk_row(order, (int)(pos & 31));
      omf[pos] = r < R ? (omega ? (float)omega[r] : 1.f) : 0.f;
    }
  }
  alpha[(int64_t)p * ldb + pos] = (float)a;
}

// Kernel 2: part[sp][a][n] (+)= sum over the split's rows of X[r][a] G'[r][n].  One workgroup of NW
// waves covers NW MI 16-row blocks of the output (all of d up to 8 x 48) for a 128-column tile;
// each wave owns MI of them, its X^T blocks straight from memory to registers, while G' is formed
// once per workgroup: 16-column blocks wave, wave + NW of each 32-row stage, G and h of the next
// stage in flight during the stage's MFMAs, through kPkBufs LDS buffers.  What bounds it: as
// k_pk_xv; G is read from memory once.
// PART: the pairs of column blocks beyond the tile's width are left out; a branch at every pair costs the
// full tiles 5 to 9% (FP32, three blocks a wave: d = 383, c = 200, s = 10, N = 60,200 843 -> 915 us), so
// that form serves where it leaves out a tenth of the pairs or more.
template <int AR, int MI, int TASKS, bool WIN, bool PART>
__global__ __launch_bounds__(64 * kPkMaxWaves, 2) void k_pk_xtg(
    const float* __restrict__ XTp, int nab, int d, const float* __restrict__ G, int64_t nrb,
    PkCols cols, const float* __restrict__ HT, int64_t ldh,
    const float* __restrict__ alpha, const float* __restrict__ omf, int64_t ldb, int64_t R,
    int64_t rows_per_split, int nmt, float* __restrict__ part, int64_t part_stride, int accumulate,
    Skip skip) {
  if (skip_now(skip)) return;
  extern __shared__ __align__(16) unsigned char pk_lds[];
  float* Bs = reinterpret_cast<float*>(pk_lds);   // [3][8][2][1 KB]
  constexpr int order = pk_order<AR, WIN>();
  const int tid = threadIdx.x, lane = tid & 63, NW = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, g = lane >> 4;
  const int nct = cols.tiles(), c = cols.c, SC = cols.SC;
  const unsigned lid = pk_lid(blockIdx.x, gridDim.x);
  const int mt = nmt == 1 ? 0 : (int)(lid % (unsigned)nmt);
  const unsigned rest = nmt == 1 ? lid : lid / (unsigned)nmt;
  const int sp = (int)(rest / (unsigned)nct);
  const int ct = (int)(rest - (unsigned)sp * nct);
  const int64_t rb = (int64_t)sp * rows_per_split;
  const int64_t re = rb + rows_per_split < R ? rb + rows_per_split : R;
  const int ab0 = (mt * NW + wave) * MI;            // the wave's first 16-row block of the output
  int n0, width;
  cols.tile(ct, n0, width);

  f32x4 acc[MI][8];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // G' tasks: column block cb = wave + NW t (t < TASKS, NW TASKS = 8); the lane's column, its class
  // row of H^T and its probe's alpha are fixed (columns beyond the tile's width read its first one:
  // only dropped outputs see them)
  const float* hp[TASKS];
  const float* bp[TASKS];
#pragma unroll
  for (int t = 0; t < TASKS; ++t) {
    const int m = 16 * (wave + NW * t) + li;
    const int n = n0 + (m < width ? m : 0), p = n / c;
    hp[t] = HT + (int64_t)(n - p * c) * ldh + 4 * g;
    bp[t] = alpha + (int64_t)p * ldb + 4 * g;
  }
  const float* gp = G + (int64_t)ct * nrb * 2048;   // uniform
  const float* op = omf + 4 * g;
  f4 gv[TASKS][2], hv[TASKS][2], bv[TASKS][2], ov[2];
  auto load_a = [&](f4 (&r)[MI][2], int64_t kb) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int ab = ab0 + i < nab ? ab0 + i : nab - 1;   // clamped blocks: dropped outputs
#pragma unroll
      for (int h = 0; h < 2; ++h)
        r[i][h] = reinterpret_cast<const f4*>(XTp + (kb * nab + ab) * 512 + h * 256)[lane];
    }
  };
  auto load_g = [&](int64_t kb) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if constexpr (!WIN) ov[q] = *reinterpret_cast<const f4*>(op + 32 * kb + 16 * q);
#pragma unroll
      for (int t = 0; t < TASKS; ++t) {
        gv[t][q] =
            reinterpret_cast<const f4*>(gp + ((2 * kb + q) * 8 + wave + NW * t) * 256)[lane];
        hv[t][q] = *reinterpret_cast<const f4*>(hp[t] + 32 * kb + 16 * q);
        bv[t][q] = *reinterpret_cast<const f4*>(bp[t] + 32 * kb + 16 * q);
      }
    }
  };
  // rows at or beyond re (only in the split's last stage) become zero in both operands
  auto store_g = [&](int64_t kb, int buf) {
#pragma unroll
    for (int t = 0; t < TASKS; ++t) {
      f4 y[2];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          y[q][v] = (gv[t][q][v] - bv[t][q][v]) * hv[t][q][v];
          if constexpr (!WIN) y[q][v] *= ov[q][v];
        }
      if (32 * kb + 32 > re) {
        const int lim = (int)(re - 32 * kb);
#pragma unroll
        for (int q = 0; q < 2; ++q)
          y[q] = pk_keep<false>(y[q], lim, [&](int v) { return pk_row(order, 16 * q + 4 * g + v); });
      }
      f4 o[2];
      pk_parts_of<AR>(y, o);
#pragma unroll
      for (int p = 0; p < 2; ++p)
        *reinterpret_cast<f4*>(Bs + buf * kPkBuf + ((wave + NW * t) * 2 + p) * 256 + lane * 4) = o[p];
    }
  };
  auto mask_a = [&](f4 (&r)[MI][2], int64_t kb) {
    if (32 * kb + 32 <= re) return;
    const int lim = (int)(re - 32 * kb);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        r[i][h] = pk_keep<AR == kPkB2>(r[i][h], lim, [&](int u) {
          return pk_row(order, AR == kPkB2 ? 16 * (u >> 2) + 4 * g + (u & 3) : 16 * h + 4 * g + u);
        });
  };
  f4 bu[2][2][2], r0[MI][2], r1[MI][2];   // the row operands as loaded, two sets in turn
  const int64_t kb0 = rb >> 5, kb1 = re > rb ? (re + 31) >> 5 : kb0, last = kb1 - 1;
  auto at = [&](int64_t kb) { return kb < last ? kb : last; };   // past the last stage: it again
  if (kb1 > kb0) {
    load_g(kb0);
    store_g(kb0, 0);
    load_g(at(kb0 + 1));
    store_g(at(kb0 + 1), 1);
    load_g(at(kb0 + 2));
    load_a(r0, kb0);
  }
  __syncthreads();
  pk_read(bu[0], Bs, 0, lane);
  // a wave without an output block only forms G'; units with a column of the tile (both uniform)
  const bool live = ab0 < nab;
  const int units = live ? (width + 31) >> 5 : 0;
  int rd = 0, nx = 1, wr = 2;
  // one stage with the operand a; the next stage's raw operand is loaded into r
  auto stage = [&](const f4 (&a)[MI][2], f4 (&r)[MI][2], int64_t kb) {
    const float* b = Bs + rd * kPkBuf;
    load_a(r, at(kb + 1));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u < 3)
        pk_read(bu[(u + 1) & 1], b, 2 * u + 2, lane);
      else
        pk_read(bu[0], Bs + nx * kPkBuf, 0, lane);
      pk_order_fence();
      if (PART ? u < units : live) pk_unit<AR, MI>(a, bu[u & 1], 2 * u, acc);
      pk_order_fence();
      if (u == 0) {   // G' two stages ahead; its next values are loaded as soon as it is stored
        store_g(at(kb + 2), wr);
        load_g(at(kb + 3));
      }
    }
    const int t = rd;
    rd = nx;
    nx = wr;
    wr = t;
    __syncthreads();
  };
  int64_t kb = kb0;
  for (; kb + 1 < kb1; kb += 2) {
    stage(r0, r1, kb);
    mask_a(r1, kb + 1);
    stage(r1, r0, kb + 1);
  }
  if (kb < kb1) {
    mask_a(r0, kb);
    stage(r0, r1, kb);
  }

  // the split's partial output: lane (g, li) of block (i, j) holds rows a = 16 (ab0 + i) + 4 g + v
  // of its column; earlier chunks' partials of one row block are loaded together, then added
  float* out = part + (int64_t)sp * part_stride;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    float prev[8][4];
    if (accumulate) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int aa = 16 * (ab0 + i) + 4 * g + v, m = 16 * j + li;
          prev[j][v] = out[aa < d && m < width ? (int64_t)aa * SC + n0 + m : 0];
        }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) prev[j][v] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int aa = 16 * (ab0 + i) + 4 * g + v, m = 16 * j + li;
        if (aa < d && m < width) out[(int64_t)aa * SC + n0 + m] = prev[j][v] + acc[i][j][v];
      }
  }
}

// Packed rows: chunk of packed position q, and the row that position holds (N or more: padding).
struct PkRows {
  int64_t N, chunk, cp;   // rows, rows per chunk, packed rows per chunk (whole tiles)
  int order;
  __device__ __forceinline__ int64_t row(int64_t q) const {
    const int64_t ch = q / cp, l = q - ch * cp;
    const int64_t r = (l & ~(int64_t)31) + pk_row(order, (int)(l & 31));
    return r < chunk && ch * chunk + r < N ? ch * chunk + r : N;
  }
};

// The two halves of an operand block from its lane's values: FP32 half h element q = val(h, q) of
// pk_k32, bf16x3 planes of val8(u).
template <bool B2, typename F>
__device__ __forceinline__ void pk_pack_block(float* __restrict__ dst, int lane, F val) {
  f4 y[2], o[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 4; ++q) y[h][q] = val(h, q);
  pk_parts_of<B2 ? kPkB2 : kPkF32>(y, o);
#pragma unroll
  for (int h = 0; h < 2; ++h) *reinterpret_cast<f4*>(dst + h * 256 + lane * 4) = o[h];
}

// X blocks: one wave per (row block, k block); padding rows and k at or beyond d are zero.
template <bool B2>
__global__ __launch_bounds__(256) void k_pk_pack_x(const float* __restrict__ X, PkRows rows, int d,
                                                   int nkb, int64_t blocks,
                                                   float* __restrict__ Xp) {
  const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= blocks) return;
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int64_t r = rows.row((b / nkb) * 16 + li);
  const int k0 = (int)(b % nkb) * 32;
  pk_pack_block<B2>(Xp + b * 512, lane, [&](int h, int q) {
    const int k = k0 + (B2 ? 8 * g + 4 * h + q : pk_k32(rows.order, h, g, q));
    return r < rows.N && k < d ? X[r * d + k] : 0.f;
  });
}

// X^T blocks: one wave per (32-row block, a block).
template <bool B2>
__global__ __launch_bounds__(256) void k_pk_pack_xt(const float* __restrict__ X, PkRows rows,
                                                    int d, int nab, int64_t blocks,
                                                    float* __restrict__ XTp) {
  const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= blocks) return;
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int a = (int)(b % nab) * 16 + li;
  const int64_t q0 = (b / nab) * 32;
  pk_pack_block<B2>(XTp + b * 512, lane, [&](int h, int q) {
    const int64_t r = rows.row(q0 + 16 * h + 4 * g + q);
    return r < rows.N && a < d ? X[r * d + a] : 0.f;
  });
}

// H^T (c x ldh) in position order, padding zero.
__global__ __launch_bounds__(256) void k_pk_pack_h(const float* __restrict__ H, PkRows rows, int c,
                                                   float* __restrict__ HT, int64_t ldh) {
  __shared__ float tile[32][33];
  const int64_t q0 = (int64_t)blockIdx.x * 32;
  const int k0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int q = ty; q < 32; q += 8) {
    const int64_t r = rows.row(q0 + q);
    tile[q][tx] = r < rows.N && k0 + tx < c ? H[r * c + k0 + tx] : 0.f;
  }
  __syncthreads();
  for (int q = ty; q < 32; q += 8)
    if (k0 + q < c) HT[(int64_t)(k0 + q) * ldh + q0 + tx] = tile[tx][q];
}

// V blocks of a probe block B (d x SC row-major): one wave per (column tile, k block, column
// block); columns beyond the tile's width and k at or beyond d are zero.
template <int AR>
__global__ __launch_bounds__(256) void k_pk_pack_v(const float* __restrict__ B, int d, PkCols cols,
                                                   int order, int nkb, int64_t blocks,
                                                   float* __restrict__ Vp, Skip skip) {
  if (skip_now(skip)) return;
  const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= blocks) return;
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int64_t tk = b >> 3;
  int n0, width;
  cols.tile((int)(tk / nkb), n0, width);
  const int m = (int)(b & 7) * 16 + li, k0 = (int)(tk % nkb) * 32;
  f4 y[2], o[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + (AR == kPkB2 ? 8 * g + 4 * h + q : pk_k32(order, h, g, q));
      y[h][q] = m < width && k < d ? B[(int64_t)k * cols.SC + n0 + m] : 0.f;
    }
  pk_parts_of<AR>(y, o);
#pragma unroll
  for (int p = 0; p < 2; ++p)
    *reinterpret_cast<f4*>(Vp + (b * 2 + p) * 256 + lane * 4) = o[p];
}

// g_r = -(1/s) sum over column tiles (in order) of the tile's row dot product.
__global__ __launch_bounds__(256) void k_pk_grad_sum(const double* __restrict__ dpart, int64_t R,
                                                     int ntiles, int s, double* __restrict__ g) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  double q = 0.0;
  for (int t = 0; t < ntiles; ++t) q += dpart[(int64_t)t * R + r];
  g[r] = -q / s;
}

// Geometry of a context's packed operands.
struct PkGeom {
  bool b2;          // bf16x3 context
  bool win;         // windows form of the row step
  int order;        // PkOrder
  int nkb, nab;
  int64_t nch, cp;  // row chunks, packed rows per chunk
  PkRows rows;
};
PkGeom pk_geom(const Ctx* x) {
  PkGeom q;
  q.b2 = x->prec == FIRAL_BF16X3;
  q.win = pk_windows(x->prec, x->d, x->c);
  q.order = q.b2 ? kPkRow8 : q.win ? kPkRowId : kPkRowQ;
  q.nkb = (int)cdiv(x->d, 32);
  q.nab = (int)cdiv(x->d, 16);
  q.nch = cdiv(x->N, x->chunk_rows);
  q.cp = cdiv(x->chunk_rows, kPkT) * kPkT;
  q.rows = PkRows{x->N, x->chunk_rows, q.cp, q.order};
  return q;
}
PkCols pk_cols(const Ctx* x, int s, bool win) {
  return PkCols{x->c, s, s * x->c, win ? (int)cdiv(x->c, kPkT) : 0};
}

// One call's view of a row chunk: packed operands at the chunk, its rows, the workspace.
struct PkChunk {
  Ctx* x;
  const PkGeom& q;
  PkCols cols;
  int64_t ch, R, Rp;
  const double* omega;   // at the chunk, or null
  Skip skip;
  hipStream_t st;
};

template <int AR, int MODE>
int pk_xv_launch(const PkChunk& k, bool prof, const float* Vp) {
  Ctx* x = k.x;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (prof) FIRAL_CHECK(prof_pair(x, FIRAL_PROF_PRODUCT, &e0, &e1));
  const unsigned nwg = (unsigned)(k.Rp / kPkT * k.cols.tiles());
  hipExtLaunchKernelGGL((k_pk_xv<AR, MODE>), dim3(nwg), dim3(256),
                        (uint32_t)pk_xv_lds<MODE>(), k.st, e0, e1, 0u,
                        (const float*)x->Xpk + k.ch * (k.q.cp / 16) * k.q.nkb * 512, k.q.nkb, k.R,
                        Vp, k.cols, (const float*)x->HTf + k.ch * k.q.cp, x->ldn,
                        k.omega, (float*)x->G, k.Rp / 16, x->pk_apart, k.Rp,
                        (const float*)x->pk_alpha, x->gpart, k.skip);
  FIRAL_LAUNCHED();
  return FIRAL_OK;
}

int pk_alpha_launch(const PkChunk& k) {
  k_pk_alpha<<<dim3((unsigned)cdiv(k.Rp, 256), (unsigned)k.cols.s), 256, 0, k.st>>>(
      k.x->pk_apart, k.cols, k.Rp, k.Rp, k.R, k.q.order, k.omega, k.x->pk_alpha, k.x->pk_om,
      k.skip);
  FIRAL_LAUNCHED();
  return FIRAL_OK;
}

// Output row tile of a second-contraction workgroup: nw waves of mi 16-row blocks, nmt tiles.  Three
// forms: 8 waves of three or of two blocks, one workgroup a CU, and 4 waves of two, two a CU; the split
// sums are the same in all.  The form with the least time by this model, in 1/20 of a block's stage on
// one SIMD: rounds of workgroups over the device, each the stages of a split (114, 80 and 74 a stage,
// windows 100; bf16x3 105, 80 and 88, 100; for 4 waves that have their CU alone half of it) and a start
// (200, for 4 waves 240).  Fitted to 440 shapes (d = 100 .. 768, SC = 35 .. 2100, 3,000 and
// 30,000 rows; 0.3% above the best of the three in the mean).  FP32 products, three blocks from d = 257
// and two below -> this: d = 257, SC = 35, N = 30,000 151 -> 78 us; d = 256, SC = 1600 611 -> 569 us; d =
// 512, SC = 2100 1898 -> 1612 us.
struct PkTile {
  int mi, nw, nmt;
};
PkTile pk_tile(const Ctx* x, const PkGeom& q, int nct, int S, int64_t rows) {
  const int64_t stages = cdiv(cdiv(rows, S), 32), splits = cdiv(rows, 32 * stages);
  const int64_t n_cu = std::max(1, x->n_cu);
  PkTile best = {};
  int64_t least = 0;
  for (int form = 0; form < 3; ++form) {
    PkTile t = {form == 0 ? 3 : 2, form == 2 ? kPkMaxWaves / 2 : kPkMaxWaves, 0};
    t.nmt = (int)cdiv(q.nab, t.mi * t.nw);
    const int64_t wgs = (int64_t)t.nmt * nct * splits;
    const bool alone = form < 2 || wgs <= n_cu;
    const int64_t four = q.win ? 100 : q.b2 ? 88 : 74;
    const int64_t unit = form == 0 ? (q.b2 ? 105 : 114) : form == 1 ? 80 : four / (alone ? 2 : 1);
    const int64_t start = form < 2 ? 200 : 240;
    const int64_t time = cdiv(wgs, form < 2 ? n_cu : 2 * n_cu) * (stages * unit + start);
    if (form == 0 || time < least) {
      best = t;
      least = time;
    }
  }
  return best;
}

template <int AR, int MI, int TASKS, bool WIN, bool PART>
int pk_xtg_launch(const PkChunk& k, const PkTile& t, int S) {
  Ctx* x = k.x;
  const int64_t rps = cdiv(cdiv(k.R, S), 32) * 32;   // splits start on whole stages
  constexpr size_t lds = kPkBufs * kPkBuf * 4;   // below the 64 KB that need no attribute, as above
  hipEvent_t e0, e1;
  FIRAL_CHECK(prof_pair(x, FIRAL_PROF_PRODUCT_T, &e0, &e1));
  hipExtLaunchKernelGGL((k_pk_xtg<AR, MI, TASKS, WIN, PART>),
                        dim3((unsigned)((int64_t)t.nmt * k.cols.tiles() * S)), dim3(64 * t.nw),
                        (uint32_t)lds, k.st, e0, e1, 0u,
                        (const float*)x->XTpk + k.ch * (k.q.cp / 32) * k.q.nab * 512, k.q.nab,
                        x->d, (const float*)x->G, k.Rp / 16, k.cols,
                        (const float*)x->HTf + k.ch * k.q.cp, x->ldn, (const float*)x->pk_alpha,
                        (const float*)x->pk_om, k.Rp, k.R, rps, t.nmt, (float*)x->part,
                        (int64_t)x->d * k.cols.SC, (int)(k.ch > 0), k.skip);
  FIRAL_LAUNCHED();
  return FIRAL_OK;
}

template <int AR, bool WIN, bool PART>
int pk_xtg_form(const PkChunk& k, const PkTile& t, int S) {
  if (t.nw < kPkMaxWaves) return pk_xtg_launch<AR, 2, 2, WIN, PART>(k, t, S);
  if (t.mi == 2) return pk_xtg_launch<AR, 2, 1, WIN, PART>(k, t, S);
  return pk_xtg_launch<AR, 3, 1, WIN, PART>(k, t, S);
}

template <int AR>
int pk_pack_v(const Ctx* x, const PkGeom& q, const PkCols& cols, const float* B, float* Vp,
              Skip skip, hipStream_t st) {
  const int64_t blocks = (int64_t)cols.tiles() * q.nkb * 8;
  k_pk_pack_v<AR><<<(unsigned)cdiv(blocks, 4), 256, 0, st>>>(B, x->d, cols, q.order, q.nkb, blocks,
                                                             Vp, skip);
  FIRAL_LAUNCHED();
  return FIRAL_OK;
}

// Row splits of the second contraction, which fix the rounding: flat, enough for several rounds of
// 128 x 128 output tiles; windows, the count with the least time in rounds over the device's slots of
// the workgroups that the row-tiled form of that shape has.
int pk_splits(const Ctx* x, const PkGeom& q, int s) {
  const int64_t cap = (int64_t)x->max_splits * x->s_max / s, nmt = cdiv(x->d, kPkT);
  if (!q.win) {
    const int64_t tiles = nmt * cdiv((int64_t)s * x->c, kPkT);
    return (int)std::max<int64_t>(1, std::min<int64_t>({cdiv(4096, tiles), cap, 256}));
  }
  const int64_t nct = s * cdiv(x->c, kPkT);
  const bool one = nmt == 2 || nmt == 3;
  const int64_t tiles = one ? nct : nmt * nct;
  const int64_t slots = (int64_t)(one ? 1 : 2) * std::max(1, x->n_cu);
  const int64_t hi =
      std::max<int64_t>(1, std::min<int64_t>({cap, 256, cdiv(x->chunk_rows, 256)}));
  int S = 1;
  for (int64_t t = 2; t <= hi; ++t)   // rounds / S, compared as cross products
    if (cdiv(tiles * t, slots) * S < cdiv(tiles * S, slots) * t) S = (int)t;
  return S;
}

template <int AR, bool WIN>
int hvp_pk_t(Ctx* x, const PkGeom& q, const double* omega, int64_t n_rows, double shift,
             const float* B, float* out, int s, Skip skip, hipStream_t st) {
  const int d = x->d, c = x->c, SC = s * c;
  const PkCols cols = pk_cols(x, s, WIN);
  float* Vp = (float*)x->Vpk;
  if (n_rows > 0) FIRAL_CHECK(pk_pack_v<AR>(x, q, cols, B, Vp, skip, st));
  const int S = pk_splits(x, q, s);
  const PkTile t =
      pk_tile(x, q, cols.tiles(), S, std::max<int64_t>(1, std::min(x->chunk_rows, n_rows)));
  for (int64_t ch = 0; ch * x->chunk_rows < n_rows; ++ch) {
    const int64_t r0 = ch * x->chunk_rows, R = std::min<int64_t>(x->chunk_rows, n_rows - r0);
    const PkChunk k{x, q, cols, ch, R, cdiv(R, kPkT) * kPkT, omega ? omega + r0 : nullptr, skip,
                    st};
    if constexpr (WIN)
      FIRAL_CHECK((pk_xv_launch<AR, kPkWin>(k, true, Vp)));
    else if (c <= kPkT)
      FIRAL_CHECK((pk_xv_launch<AR, kPkFlat>(k, true, Vp)));
    else
      FIRAL_CHECK((pk_xv_launch<AR, kPkFlatX>(k, true, Vp)));
    FIRAL_CHECK(pk_alpha_launch(k));
    FIRAL_CHECK((cols.part() ? pk_xtg_form<AR, WIN, true>(k, t, S)
                             : pk_xtg_form<AR, WIN, false>(k, t, S)));
  }
  return reduce_parts_launch<float>((const float*)x->part, (int64_t)d * SC, n_rows > 0 ? S : 0,
                                    shift, B, out, skip, st);
}

template <int AR>
int grad_pk_t(Ctx* x, const PkGeom& q, const float* U, const float* W, int s, double* g,
              hipStream_t st) {
  const int c = x->c;
  const PkCols cols = pk_cols(x, s, false);
  float* Wp = (float*)x->Vpk;
  float* Up = Wp + (int64_t)pk_cols(x, x->s_max, false).tiles() * q.nkb * 8 * 512;
  FIRAL_CHECK(pk_pack_v<AR>(x, q, cols, W, Wp, skip_none(), st));
  FIRAL_CHECK(pk_pack_v<AR>(x, q, cols, U, Up, skip_none(), st));
  for (int64_t ch = 0; ch * x->chunk_rows < x->n_pool; ++ch) {
    const int64_t r0 = ch * x->chunk_rows, R = std::min<int64_t>(x->chunk_rows, x->n_pool - r0);
    const PkChunk k{x, q, cols, ch, R, cdiv(R, kPkT) * kPkT, nullptr, skip_none(), st};
    if (c <= kPkT)
      FIRAL_CHECK((pk_xv_launch<AR, kPkFlat>(k, false, Wp)));
    else
      FIRAL_CHECK((pk_xv_launch<AR, kPkFlatX>(k, false, Wp)));
    FIRAL_CHECK(pk_alpha_launch(k));
    FIRAL_CHECK((pk_xv_launch<AR, kPkDot>(k, false, Up)));
    k_pk_grad_sum<<<(unsigned)cdiv(R, 256), 256, 0, st>>>(x->gpart, R, cols.tiles(), s, g + r0);
    FIRAL_LAUNCHED();
  }
  return FIRAL_OK;
}

template <bool B2>
int pk_pack_ctx(Ctx* x, const PkGeom& q, hipStream_t st) {
  const int64_t Np = q.nch * q.cp, bx = Np / 16 * q.nkb, bt = Np / 32 * q.nab;
  k_pk_pack_x<B2><<<(unsigned)cdiv(bx, 4), 256, 0, st>>>((const float*)x->X, q.rows, x->d, q.nkb,
                                                         bx, (float*)x->Xpk);
  FIRAL_LAUNCHED();
  k_pk_pack_xt<B2><<<(unsigned)cdiv(bt, 4), 256, 0, st>>>((const float*)x->X, q.rows, x->d, q.nab,
                                                          bt, (float*)x->XTpk);
  FIRAL_LAUNCHED();
  const dim3 grid((unsigned)(Np / 32), (unsigned)cdiv(x->c, 32));
  k_pk_pack_h<<<grid, 256, 0, st>>>((const float*)x->H, q.rows, x->c, (float*)x->HTf, x->ldn);
  FIRAL_LAUNCHED();
  return FIRAL_OK;
}

}  // namespace

bool pk_windows(int prec, int d, int c) {
  return d > 128 && c > kPkT && d % (prec == FIRAL_BF16X3 ? 8 : 4) == 0;
}

PkSizes pk_sizes(const Ctx* x) {
  const PkGeom q = pk_geom(x);
  PkSizes z;
  const int64_t Np = q.nch * q.cp;
  // the flat and the windows form share the buffers
  const PkCols cf = pk_cols(x, x->s_max, false), cw = pk_cols(x, x->s_max, true);
  const int64_t nct = q.win ? std::max(cf.tiles(), cw.tiles()) : cf.tiles();
  z.ldn = Np;
  z.x = (size_t)(Np / 16) * q.nkb * 2048;
  z.xt = (size_t)(Np / 32) * q.nab * 2048;
  z.ht = (size_t)Np * x->c * 4;
  // two blocks of V (the gradient's W and U)
  z.v = (size_t)2 * nct * q.nkb * 8 * 2048;
  z.g = (size_t)nct * kPkT * q.cp * 4;
  z.apart = (size_t)(nct + x->s_max) * q.cp * 8;
  z.alpha = (size_t)x->s_max * q.cp * 4;
  z.om = (size_t)q.cp * 4;
  z.dpart = (size_t)cf.tiles() * q.cp * 8;
  return z;
}

int pk_prepare_ctx(Ctx* x, hipStream_t st) {
  const PkGeom q = pk_geom(x);
  return q.b2 ? pk_pack_ctx<true>(x, q, st) : pk_pack_ctx<false>(x, q, st);
}

// A bf16x3 context's packed operands are bf16 planes: its FP32 products (precise) are row-tiled.  So are
// those of FP32 contexts with d <= 128 (and wide probes) up to 2048 rows, where the two launches more
// of the packed form show: d = 98, c = 500, s = 7, N = 408 97 us, row-tiled 80; d = 91, c = 300, N = 1182
// 72, 63; at 2,500 rows and more the packed form is the faster one (d = 89, c = 160, s = 8, N = 2600 59,
// row-tiled 64).
bool hvp_pk_applies(const Ctx* x, int64_t n_rows, bool precise) {
  if (!x->use_pk) return false;
  if (x->prec == FIRAL_BF16X3) return !precise;
  return x->d > 128 || n_rows > 2048;
}

int hvp_pk_launch(Ctx* x, const double* omega, int64_t n_rows, double shift, const float* B,
                  float* out, int s, Skip skip, hipStream_t st) {
  const PkGeom q = pk_geom(x);
#define FIRAL_PK_HVP(AR)                                                              \
  return q.win ? hvp_pk_t<AR, true>(x, q, omega, n_rows, shift, B, out, s, skip, st) \
               : hvp_pk_t<AR, false>(x, q, omega, n_rows, shift, B, out, s, skip, st)
  if (q.b2) FIRAL_PK_HVP(kPkB2);
  FIRAL_PK_HVP(kPkF32);
#undef FIRAL_PK_HVP
}

bool grad_pk_applies(const Ctx* x) {
  return x->use_pk && (x->prec == FIRAL_BF16X3 || !pk_windows(x->prec, x->d, x->c));
}

int grad_pk_launch(Ctx* x, const float* U, const float* W, int s, double* g, hipStream_t st) {
  const PkGeom q = pk_geom(x);
  return q.b2 ? grad_pk_t<kPkB2>(x, q, U, W, s, g, st) : grad_pk_t<kPkF32>(x, q, U, W, s, g, st);
}

}  // namespace firal
