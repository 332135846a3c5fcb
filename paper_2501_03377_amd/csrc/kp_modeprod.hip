// Mode products of the pseudoinverse preconditioner (Algs. 6 and 7, Sec. 4.3.3)
// on the gfx950 matrix cores.
//
// Z = (V_x, V_y, V_z | G .* (V_x^T, V_y^T, V_z^T | R)).  Every l-mode product
// is applied as one GEMM that contracts the *contiguous* axis of its input:
//     C[r][n] = sum_k X[r][k] B[k][n],    X viewed as [A0][A1][K] -> rows r,
// and writes C transposed, Y[n][r], i.e. the layout [K'][A0][A1]: the
// transformed axis moves to the front.  Three such products return the
// original layout, so the sequence (3D; grids stored [z][y][x], x fastest)
//   [z][y][x] -x->  [x'][z][y] -y-> [y'][x'][z] -z,G-> [z'][y'][x']
//             -x->  [x][z'][y'] -y-> [y][x][z']  -z->  [z][y][x]
// contracts x, y, z forward, applies the Hadamard factor G of eq. (4.6) in the
// third product's epilogue, and contracts x, y, z backward (2D: x, y+G, x, y).
// The mode products commute (Sec. 2.2), so this order is the paper's operator.
//
// This file: the BF16 products (plain, and split in three terms) and the order
// of the products; the FP64 and FP32 ones are in kp_fold.hip, the int8 split
// ones in kp_oz.hip.
//
// Operands (BF16).  B (V_l forward, V_l^T backward) is packed at plan time in
// fragment order and streamed through a double-buffered LDS chunk shared by
// the block's four waves; each wave loads its own rows of X straight into
// registers (CH consecutive k per lane, 16-byte loads).  MFMA:
// v_mfma_f32_16x16x32_bf16 with FP32 accumulation.  Lane l supplies row (X) /
// column (B) l%16 and the k values CH*(l/16) .. +CH-1 of each k-block; output
// item v of lane l is column l%16 and row 4*(l/16)+v.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "kp_common.h"
#include "kp_internal.h"

namespace kp {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));   // one 16-byte unit

template <int PREC> struct MT;
template <> struct MT<PREC_BF16> {
  using tc = __bf16; using acc = f4;
  static constexpr int CH = 8, NV = 1, STEPS = 1;
  struct chunk { bf8 v; };
  static __device__ __forceinline__ acc mma(const chunk& a, const chunk& b, acc c, int) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};

// FP32-accurate products on the BF16 matrix cores: a chunk holds the three
// BF16 terms of 8 values (x = x1 + x2 + x3); step s accumulates the product
// of data term split_a(s) and operator term split_b(s), the six pairs with
// i + j <= 2 (0-based), largest first.
constexpr int split_a(int s) { return (s == 2 || s == 4) ? 1 : (s == 5 ? 2 : 0); }
constexpr int split_b(int s) { return (s == 1 || s == 4) ? 1 : (s == 3 ? 2 : 0); }
template <> struct MT<PREC_BF16X6> {
  using tc = float; using acc = f4;
  static constexpr int CH = 8, NV = 3, STEPS = 6;
  struct chunk { bf8 p[3]; };
  static __device__ __forceinline__ acc mma(const chunk& a, const chunk& b, acc c, int s) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[split_a(s)], b.p[split_b(s)], c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};

// What the FP64 and FP32 products (kp_fold.hip) and the int8 split products
// (kp_oz.hip) keep between products.
template <> struct MT<PREC_F64> {
  using tc = double;
};
template <> struct MT<PREC_F32> {
  using tc = float;
};
template <> struct MT<PREC_I8X7> {
  using tc = double;
};
template <> struct MT<PREC_I8X6> {
  using tc = double;
};

// Block = WR x WC waves (WR = 4 row groups, WC column groups); each wave owns
// WM row fragments x WN column fragments of 16 x 16.
constexpr int WR = 4;

template <int PREC>
__device__ __forceinline__ typename MT<PREC>::tc to_tc(double x) {
  if constexpr (PREC == PREC_BF16) return (__bf16)(float)x;
  else return (typename MT<PREC>::tc)x;
}

// ---- one lane's CH consecutive k values of one row --------------------------
// Loaded raw (source type) into a register ring and converted only when the
// MFMA needs them, so that no arithmetic waits on a load in flight.  Lanes
// past the end of the row (k0 >= K, and rows past the end, which arrive with
// k0 = K) read the row's last CH values instead: the packed operator is zero
// for k >= K, so they add nothing (both are finite data of the same grid).
// VEC: the row length is a multiple of CH (16-byte loads); else CH scalar
// loads.
template <int PREC, class Ti> struct XRaw { Ti v[MT<PREC>::CH]; };

template <int PREC, class Ti, bool VEC>
__device__ __forceinline__ XRaw<PREC, Ti> load_raw(const Ti* __restrict__ row, int k0, int K) {
  constexpr int CH = MT<PREC>::CH;
  XRaw<PREC, Ti> x;
  if constexpr (VEC) {
    const Ti* src = row + (k0 < K ? k0 : K - CH);
    static_assert((CH * sizeof(Ti)) % 16 == 0, "whole 16-byte units");
#pragma unroll
    for (int q = 0; q < (int)(CH * sizeof(Ti)) / 16; ++q) {
      const u4 u = *reinterpret_cast<const u4*>(reinterpret_cast<const char*>(src) + 16 * q);
      __builtin_memcpy(reinterpret_cast<char*>(x.v) + 16 * q, &u, 16);
    }
  } else {
#pragma unroll
    for (int s = 0; s < CH; ++s) x.v[s] = row[k0 + s < K ? k0 + s : K - 1];
  }
  return x;
}

template <int PREC, class Ti>
__device__ __forceinline__ typename MT<PREC>::chunk cvt_raw(const XRaw<PREC, Ti>& x, double scale,
                                                           bool scaled) {
  using M = MT<PREC>;
  typename M::chunk c;
  if constexpr (PREC == PREC_BF16X6) {
    // three round-to-nearest BF16 terms; each remainder is exact in FP32
#pragma unroll
    for (int s = 0; s < M::CH; ++s) {
      float f;
      if constexpr (sizeof(Ti) == 8) f = (float)(scaled ? x.v[s] * scale : x.v[s]);
      else f = x.v[s];
      const __bf16 t1 = (__bf16)f;
      const float r1 = f - (float)t1;
      const __bf16 t2 = (__bf16)r1;
      const float r2 = r1 - (float)t2;
      c.p[0][s] = t1;
      c.p[1][s] = t2;
      c.p[2][s] = (__bf16)r2;
    }
  } else if constexpr (std::is_same<Ti, typename M::tc>::value) {
    __builtin_memcpy(&c, &x, sizeof(c));
  } else {
#pragma unroll
    for (int s = 0; s < M::CH; ++s) {
      const double d = to_double(x.v[s]);
      c.v[s] = to_tc<PREC>(scaled ? d * scale : d);
    }
  }
  return c;
}

template <int PREC>
__device__ __forceinline__ typename MT<PREC>::chunk load_b(const u4* __restrict__ l, int g,
                                                          int c, int CB) {
  using M = MT<PREC>;
  typename M::chunk b;
  static_assert(sizeof(b) == 16 * M::NV, "a chunk is NV 16-byte units");
#pragma unroll
  for (int h = 0; h < M::NV; ++h) {
    const u4 u = l[(g * M::NV + h) * CB + c];
    __builtin_memcpy(reinterpret_cast<char*>(&b) + 16 * h, &u, 16);
  }
  return b;
}

// ---------------------------------------------------------------------------
// One mode product for `batch` right-hand sides.
//   Bpk   packed operator: 16-byte unit (kb, g, h, n) at ((kb*4+g)*NV+h)*npk+n
//   X     input  [rhs][rows][K]  (type Ti)
//   Y     output [rhs][K][rows]  (type To): Y[n*rows + r] = sum_k X[r][k] B[k][n]
//   G epilogue (lc != nullptr): times ghat(la[r % a1] + lb[r / a1] + lc[n])
//   table epilogue (gt != nullptr): times gt[n * rows + r], a precomputed
//   factor in the output's layout (the low-rank preconditioner's G_r)
//   in_scale / out_scale: per-RHS power-of-two scale on the input / its
//   inverse on the output (low-precision range guard)
// Grid: x = row blocks * column chunks, y = right-hand side.
// ---------------------------------------------------------------------------
constexpr int group_size(int wn, int most) {
  int j = wn < most ? wn : most;
  while (wn % j != 0) --j;
  return j;
}
static_assert(group_size(6, 4) == 3 && group_size(12, 8) == 6 && group_size(16, 8) == 8, "");

template <int PREC, class Ti, class To, int WN, int WM, int WC, bool VEC>
__global__ __launch_bounds__(64 * WR * WC, WC == 1 ? 2 : 1) void mp_kernel(
    const u4* __restrict__ Bpk, int npk, int ncc, const Ti* __restrict__ X, To* __restrict__ Y,
    int K, int rows, int64_t N, const RhsState* __restrict__ st, int in_scale, int out_scale,
    const double* __restrict__ la, const double* __restrict__ lb, const double* __restrict__ lc,
    int a1, const double* __restrict__ gt) {
  using M = MT<PREC>;
  constexpr int NT = 64 * WR * WC;
  constexpr int CW = 16 * WN;                 // columns per wave
  constexpr int CB = WC * CW;                 // columns per block
  constexpr int BR = WR * 16 * WM;            // rows per block
  constexpr int CH = M::CH, NV = M::NV, KB = 4 * CH;
  constexpr int UNITS = 4 * NV * CB;          // 16-byte units per operator k-block
  // k-blocks per LDS stage (one barrier per stage), at most 32 KiB per stage
  // (two stages resident), 64 KiB for the eight-wave tiles, which run one
  // block per CU anyway.  The data rows are prefetched one stage ahead in a
  // register ring of KS k-blocks indexed by the unrolled step, so no register
  // ever moves inside the ring; larger stages prefetch further ahead.
  constexpr int SBYTES = (WC == 2 && WM < 4) ? 65536 : 32768;
  constexpr int KSL = SBYTES / (16 * UNITS) > 0 ? SBYTES / (16 * UNITS) : 1;
  constexpr int KS = KSL < 4 ? KSL : 4;
  constexpr int SUNITS = KS * UNITS;          // units per stage
  constexpr int UPT = (SUNITS + NT - 1) / NT; // units per thread per stage
  // operator fragments read per group: the largest divisor of WN whose
  // fragments take at most 32 VGPRs
  constexpr int JG = group_size(WN, PREC == PREC_BF16X6 ? 4 : 8);
  // data ring depth: KS k-blocks, halved while the raw data would take more
  // than 64 VGPRs (the FP64 sources of the first product are twice as wide)
  constexpr int RAWV = CH * (int)sizeof(Ti) / 4;
  constexpr int XD = (KS * WM * RAWV <= 64 || KS == 1) ? KS
                     : ((KS / 2) * WM * RAWV <= 64 || KS == 2) ? KS / 2 : KS / 4;
  static_assert(KS % XD == 0, "ring depth divides the stage");

  const int rhs = blockIdx.y;
  if (st && st[rhs].done) return;
  const int cc = blockIdx.x % ncc, rb = blockIdx.x / ncc;
  const int c0 = cc * CB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave % WR, wc = wave / WR;
  const int g = lane >> 4, l16 = lane & 15;
  const int rw = rb * BR + wr * WM * 16;      // this wave's first row
  const int cw = wc * CW;                     // this wave's first column in the block
  const Ti* Xb = X + (int64_t)rhs * N;
  const bool scaled = (st != nullptr) && in_scale;
  const double scale = scaled ? st[rhs].scale : 1.0;
  const int nkb = (K + KB - 1) / KB;

  __shared__ u4 lds[2][SUNITS];

  const Ti* xrow[WM];
  bool rok[WM];
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int r = rw + 16 * i + l16;
    rok[i] = r < rows;
    xrow[i] = Xb + (int64_t)(rok[i] ? r : 0) * K;
  }

  typename M::acc acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0;

  // Plain unrolled loops, no closures over these arrays: a captured array
  // gets an address and lands in scratch memory.
  u4 breg[UPT];
  XRaw<PREC, Ti> xq[XD][WM];
  constexpr bool FULL = (SUNITS % NT) == 0;
  const u4* bsrc = Bpk + c0;
  const int cmax = npk - c0;                  // packed columns left for this block
  const int nst = (nkb + KS - 1) / KS;

  // Loads stage `sg` of the operator into breg.  Every load is issued
  // unconditionally, with clamped indices, so that the compiler counts the
  // same loads in flight on every path and waits only for the ones it needs:
  // k-blocks past the end (last stage) and columns past the end (ragged last
  // column chunk) only feed accumulators that are never stored, and threads
  // past the stage size repeat the last unit (the same value to the same
  // LDS address).
#define KP_LOAD_STAGE(sg)                                                                  \
  _Pragma("unroll") for (int q = 0; q < UPT; ++q) {                                       \
    const int su = FULL ? tid + q * NT : min(tid + q * NT, SUNITS - 1);                    \
    const int kk = su / UNITS, u = su % UNITS, gh = u / CB;                                \
    const int c = min(u % CB, cmax - 1);                                                   \
    const int kbg = min((sg) * KS + kk, nkb - 1);                                          \
    breg[q] = bsrc[((int64_t)kbg * 4 * NV + gh) * npk + c];                                \
  }
#define KP_STORE_STAGE(bf)                                                                 \
  _Pragma("unroll") for (int q = 0; q < UPT; ++q) {                                       \
    const int su = FULL ? tid + q * NT : min(tid + q * NT, SUNITS - 1);                    \
    lds[bf][su] = breg[q];                                                                 \
  }

  KP_LOAD_STAGE(0)
#pragma unroll
  for (int d = 0; d < XD; ++d) {
    const int k0 = d * KB + CH * g;
#pragma unroll
    for (int i = 0; i < WM; ++i)
      xq[d][i] = load_raw<PREC, Ti, VEC>(xrow[i], (rok[i] && d < nkb) ? k0 : K, K);
  }
  KP_STORE_STAGE(0)
  __syncthreads();

  for (int sg = 0; sg < nst; ++sg) {
    const int buf = sg & 1;
    KP_LOAD_STAGE(sg + 1)   // past the last stage: a harmless reload
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const int kb = sg * KS + kk;
      const int slot = kk % XD;
      if (KS == 1 || kb < nkb) {
        typename M::chunk xa[WM];
#pragma unroll
        for (int i = 0; i < WM; ++i) xa[i] = cvt_raw<PREC, Ti>(xq[slot][i], scale, scaled);
#pragma unroll
        for (int j0 = 0; j0 < WN; j0 += JG) {
          typename M::chunk b[JG];
#pragma unroll
          for (int jj = 0; jj < JG; ++jj)
            b[jj] = load_b<PREC>(lds[buf] + kk * UNITS, g, cw + 16 * (j0 + jj) + l16, CB);
          // consecutive MFMAs update different accumulators
#pragma unroll
          for (int s = 0; s < M::STEPS; ++s)
#pragma unroll
            for (int jj = 0; jj < JG; ++jj)
#pragma unroll
              for (int i = 0; i < WM; ++i)
                acc[i][j0 + jj] = M::mma(xa[i], b[jj], acc[i][j0 + jj], s);
        }
      }
      // this ring slot now takes k-block kb + XD
      const int kn = kb + XD;
      const int k0 = kn * KB + CH * g;
#pragma unroll
      for (int i = 0; i < WM; ++i)
        xq[slot][i] = load_raw<PREC, Ti, VEC>(xrow[i], (rok[i] && kn < nkb) ? k0 : K, K);
    }
    KP_STORE_STAGE(buf ^ 1)   // the buffer not read in this stage
    __syncthreads();
  }
#undef KP_LOAD_STAGE
#undef KP_STORE_STAGE

  // ---- epilogue: optional G factor and output scale, transposed store ------
  const double oscale = (st && out_scale) ? st[rhs].inv_scale : 1.0;
  To* Yb = Y + (int64_t)rhs * N;
  double rowsum[WM][4];
  if (lc) {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = rw + 16 * i + M::row(lane, v);
        const int rc = r < rows ? r : 0;
        rowsum[i][v] = la[rc % a1] + (lb ? lb[rc / a1] : 0.0);
      }
  }
  // Outputs of at most 4 bytes: the block's tile is staged in LDS (free after
  // the k-loop) as [column][row], then written column by column, 16 bytes a
  // thread, so that each column gets one contiguous run of BR rows instead
  // of 16-row pieces from every wave.
  constexpr int SE = 16 / (int)sizeof(To);          // elements per 16-byte chunk
  constexpr int BRP = BR + SE;                      // padded column length
  constexpr bool STG = sizeof(To) <= 4 && (size_t)CB * BRP * sizeof(To) <= sizeof(lds);
  const bool stage = STG && rows % SE == 0;
  To* stg = reinterpret_cast<To*>(&lds[0][0]);
#pragma unroll
  for (int j = 0; j < WN; ++j) {
    const int n = c0 + cw + 16 * j + l16;
    if (n >= K) continue;
    const double lcn = lc ? lc[n] : 0.0;
    To* dst = Yb + (int64_t)n * rows;
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      To out[4];
      int rr[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        rr[v] = rw + 16 * i + M::row(lane, v);
        double val = (double)acc[i][j][v];
        if (lc) {
          const double sum = rowsum[i][v] + lcn;
          // FP32 reciprocal: the low-precision preconditioner is accurate to
          // its own rounding anyway
          val = fabs(sum) < 1e-13 ? 0.0 : (double)((float)val * __frcp_rn((float)sum));
        }
        if (gt) val *= gt[(int64_t)n * rows + (rr[v] < rows ? rr[v] : 0)];
        if (out_scale) val *= oscale;
        if constexpr (sizeof(To) == 2) out[v] = (__bf16)(float)val;
        else out[v] = (To)val;
      }
      if constexpr (STG) {
        if (stage) {
          // the four rows of this lane are consecutive
          To* q = stg + (cw + 16 * j + l16) * BRP + wr * WM * 16 + 16 * i + M::row(lane, 0);
          if constexpr (sizeof(To) == 4) {
            const f4 a = {out[0], out[1], out[2], out[3]};
            *reinterpret_cast<f4*>(q) = a;
          } else {
            const bf4 a = {out[0], out[1], out[2], out[3]};
            *reinterpret_cast<bf4*>(q) = a;
          }
          continue;
        }
      }
      // the four rows of this lane are consecutive
      if ((rows & 3) == 0 && rr[3] < rows) {
        if constexpr (sizeof(To) == 8) {
          const d2 a = {out[0], out[1]}, b2 = {out[2], out[3]};
          *reinterpret_cast<d2*>(dst + rr[0]) = a;
          *reinterpret_cast<d2*>(dst + rr[0] + 2) = b2;
        } else if constexpr (sizeof(To) == 4) {
          const f4 a = {out[0], out[1], out[2], out[3]};
          *reinterpret_cast<f4*>(dst + rr[0]) = a;
        } else {
          const bf4 a = {out[0], out[1], out[2], out[3]};
          *reinterpret_cast<bf4*>(dst + rr[0]) = a;
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (rr[v] < rows) dst[rr[v]] = out[v];
      }
    }
  }
  if constexpr (STG) {
    if (stage) {
      __syncthreads();
      constexpr int CPC = BR / SE;                  // chunks per column
      const int nvalid = min(CB, K - c0);
      const int r0 = rb * BR;
      for (int c = tid; c < CB * CPC; c += NT) {
        const int col = c / CPC, part = c - col * CPC;
        const int row = r0 + part * SE;
        if (col >= nvalid || row >= rows) continue;   // (rows is a multiple of SE)
        *reinterpret_cast<u4*>(Yb + (int64_t)(c0 + col) * rows + row) =
            *reinterpret_cast<const u4*>(stg + col * BRP + part * SE);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Operator-resident variant for short contractions (K <= 128).  The whole
// packed operator of one product (at most 128 KiB) is loaded into LDS once
// per block; the block then sweeps row tiles of 64 rows x 128 columns
// (WR x WC waves, each 16 rows x 16*WN columns) with no further barrier on
// the operator.  A tile's rows are converted to the compute type, then the
// next tile's rows are requested, so their loads overlap this tile's
// products and stores.  Every output is summed over k in the same order as
// in mp_kernel (bitwise the same product).  BF16 outputs (the
// HBM-bound products) are staged in LDS as [column][64 rows] and written a
// column's 128 contiguous bytes at a time, 16 bytes a thread, instead of 8
// bytes a lane scattered over 16 columns.
template <int PREC, class Ti, class To, int WN, int WC>
__global__ __launch_bounds__(64 * WR * WC, 1) void mp_res(
    const u4* __restrict__ Bpk, int npk, const Ti* __restrict__ X, To* __restrict__ Y, int K,
    int rows, int64_t N, const RhsState* __restrict__ st, int in_scale, int out_scale,
    const double* __restrict__ la, const double* __restrict__ lb, const double* __restrict__ lc,
    int a1, const double* __restrict__ gt) {
  using M = MT<PREC>;
  constexpr int NT = 64 * WR * WC;
  constexpr int CW = 16 * WN;                 // columns per wave
  constexpr int CB = WC * CW;                 // columns per block
  static_assert(CB == 128, "one block covers the operator's 128 columns");
  constexpr int BR = WR * 16;                 // rows per tile
  constexpr int CH = M::CH, NV = M::NV, KB = 4 * CH;
  constexpr int UNITS = 4 * NV * CB;          // 16-byte units per operator k-block
  constexpr int KBMAX = 128 / KB;             // k-blocks of a 128 x 128 operator
  constexpr int JG = group_size(WN, PREC == PREC_BF16X6 ? 4 : 8);

  const int rhs = blockIdx.y;
  if (st && st[rhs].done) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave % WR, wc = wave / WR;
  const int g = lane >> 4, l16 = lane & 15;
  const int cw = wc * CW;
  const Ti* Xb = X + (int64_t)rhs * N;
  To* Yb = Y + (int64_t)rhs * N;
  const bool scaled = (st != nullptr) && in_scale;
  const double scale = scaled ? st[rhs].scale : 1.0;
  const double oscale = (st && out_scale) ? st[rhs].inv_scale : 1.0;
  const int nkb = (K + KB - 1) / KB;
  const int nrb = (rows + BR - 1) / BR;

  __shared__ u4 lds[KBMAX * UNITS];
  constexpr bool STG = sizeof(To) == 2;
  constexpr int SE = 8, BRP = BR + SE;          // elements per 16-byte chunk; padded column
  __shared__ __attribute__((aligned(16))) To stg[STG ? CB * BRP : 1];
  const bool stage = STG && rows % SE == 0;
  for (int su = tid; su < nkb * UNITS; su += NT) {
    const int kk = su / UNITS, u = su % UNITS, gh = u / CB;
    const int c = min(u % CB, npk - 1);
    lds[su] = Bpk[((int64_t)kk * 4 * NV + gh) * npk + c];
  }

  // this lane's row data of tile rb (rows past the end, and k-blocks past the
  // operator, read valid data that only feeds unused sums)
  XRaw<PREC, Ti> xq[KBMAX];
  int rb = blockIdx.x;
  {
    const int r = rb * BR + wr * 16 + l16;
    const bool ok = r < rows;
    const Ti* xr = Xb + (int64_t)(ok ? r : 0) * K;
#pragma unroll
    for (int d = 0; d < KBMAX; ++d)
      xq[d] = load_raw<PREC, Ti, true>(xr, (ok && d < nkb) ? d * KB + CH * g : K, K);
  }
  __syncthreads();

  for (; rb < nrb; rb += gridDim.x) {
    typename M::chunk xa[KBMAX];
#pragma unroll
    for (int d = 0; d < KBMAX; ++d) xa[d] = cvt_raw<PREC, Ti>(xq[d], scale, scaled);
    {
      // the next tile's rows, while this one is computed
      const int rn = rb + gridDim.x;
      const int r = rn * BR + wr * 16 + l16;
      const bool ok = rn < nrb && r < rows;
      const Ti* xr = Xb + (int64_t)(ok ? r : 0) * K;
#pragma unroll
      for (int d = 0; d < KBMAX; ++d)
        xq[d] = load_raw<PREC, Ti, true>(xr, (ok && d < nkb) ? d * KB + CH * g : K, K);
    }
    typename M::acc acc[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[j][v] = 0;
#pragma unroll
    for (int kk = 0; kk < KBMAX; ++kk) {
      if (kk < nkb) {
#pragma unroll
        for (int j0 = 0; j0 < WN; j0 += JG) {
          typename M::chunk b[JG];
#pragma unroll
          for (int jj = 0; jj < JG; ++jj)
            b[jj] = load_b<PREC>(lds + kk * UNITS, g, cw + 16 * (j0 + jj) + l16, CB);
#pragma unroll
          for (int s = 0; s < M::STEPS; ++s)
#pragma unroll
            for (int jj = 0; jj < JG; ++jj)
              acc[j0 + jj] = M::mma(xa[kk], b[jj], acc[j0 + jj], s);
        }
      }
    }

    // epilogue: optional G factor and output scale, transposed store
    const int rw = rb * BR + wr * 16;
    double rowsum[4];
    if (lc) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = rw + M::row(lane, v);
        const int rc = r < rows ? r : 0;
        rowsum[v] = la[rc % a1] + (lb ? lb[rc / a1] : 0.0);
      }
    }
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int n = cw + 16 * j + l16;
      if (n >= K) continue;
      const double lcn = lc ? lc[n] : 0.0;
      To* dst = Yb + (int64_t)n * rows;
      To out[4];
      int rr[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        rr[v] = rw + M::row(lane, v);
        double val = (double)acc[j][v];
        if (lc) {
          const double sum = rowsum[v] + lcn;
          val = fabs(sum) < 1e-13 ? 0.0 : (double)((float)val * __frcp_rn((float)sum));
        }
        if (gt) val *= gt[(int64_t)n * rows + (rr[v] < rows ? rr[v] : 0)];
        if (out_scale) val *= oscale;
        if constexpr (sizeof(To) == 2) out[v] = (__bf16)(float)val;
        else out[v] = (To)val;
      }
      if constexpr (STG) {
        if (stage) {
          // the four rows of this lane are consecutive
          To* q = stg + (cw + 16 * j + l16) * BRP + wr * 16 + M::row(lane, 0);
          *reinterpret_cast<bf4*>(q) = (bf4){out[0], out[1], out[2], out[3]};
          continue;
        }
      }
      if ((rows & 3) == 0 && rr[3] < rows) {
        if constexpr (sizeof(To) == 8) {
          const d2 a = {out[0], out[1]}, b2 = {out[2], out[3]};
          *reinterpret_cast<d2*>(dst + rr[0]) = a;
          *reinterpret_cast<d2*>(dst + rr[0] + 2) = b2;
        } else if constexpr (sizeof(To) == 4) {
          const f4 a = {out[0], out[1], out[2], out[3]};
          *reinterpret_cast<f4*>(dst + rr[0]) = a;
        } else {
          const bf4 a = {out[0], out[1], out[2], out[3]};
          *reinterpret_cast<bf4*>(dst + rr[0]) = a;
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (rr[v] < rows) dst[rr[v]] = out[v];
      }
    }
    if constexpr (STG) {
      if (stage) {
        __syncthreads();
        constexpr int CPC = BR / SE;            // 16-byte chunks per column
        const int nvalid = min(CB, K);
        for (int c = tid; c < CB * CPC; c += NT) {
          const int col = c / CPC, part = c - col * CPC;
          const int row = rw - wr * 16 + part * SE;   // the tile's first row + 8 part
          if (col >= nvalid || row >= rows) continue;  // (rows is a multiple of SE)
          *reinterpret_cast<u4*>(Yb + (int64_t)col * rows + row) =
              *reinterpret_cast<const u4*>(stg + col * BRP + part * SE);
        }
        __syncthreads();                        // the next tile stages over it
      }
    }
  }
}

// ------------------------------------------------------------------ host ----
// Tile configurations (column fragments per wave, row fragments per wave,
// column wave groups).  Block = 4 x wc waves, rows per block 64*wm, columns
// per block 16*wn*wc.  The operator packing does not depend on the choice, so
// any configuration may serve any product; the autotuner times them.
struct MpCfg { int wn, wm, wc; };
static const MpCfg kCfgs[] = {
    {1, 4, 1}, {2, 4, 1}, {3, 4, 1}, {4, 4, 1}, {6, 2, 1}, {8, 2, 1}, {12, 1, 1}, {16, 1, 1},
    {2, 4, 2}, {3, 4, 2}, {4, 2, 2}, {4, 4, 2}, {6, 2, 2}, {8, 1, 2}, {8, 2, 2}, {16, 1, 2},
    // tall tiles (FP32 and BF16 accumulators only): fewer re-reads of the operator
    {16, 2, 1}, {8, 4, 2},
    // short tiles of 128 columns: more blocks for short contractions
    {8, 1, 1}, {4, 1, 2},
    // operator-resident tiles (mp_res) of the same shapes, for K <= 128
    {8, 1, 1}, {4, 1, 2},
};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);
constexpr int kResFirst = 20;   // ids from here on are operator-resident
constexpr int kOzCfg = 13;      // the id an int8 split plan reports (its tiles follow the size)

int mp_num_configs() { return kNumCfgs; }

bool mp_config_resident(int id) { return id >= kResFirst && id < kNumCfgs; }

// Whether configuration `id` can serve a K x K operator: the operator-resident
// tiles hold at most 128 x 128.
bool mp_config_fits(int id, int K) { return !mp_config_resident(id) || K <= 128; }

// Whether a plan of `prec` accepts configuration `id`.  BF16 and BF16X6: it is
// compiled (tiles whose registers would spill are left out).  FP64 and FP32
// products choose their tiles by size: their plans accept and report the ids
// that saved choices may hold, and none changes a product.
bool mp_config_allowed(int id, int prec) {
  if (id < 0 || id >= kNumCfgs) return false;
  if (prec_int8(prec)) return id == kOzCfg;     // one kernel serves every product
  if (prec == PREC_F64) return !(id == 3 || id == 7 || id == 11 || (id >= 15 && id <= 17));
  if (prec == PREC_BF16) return id != 16;
  if (prec == PREC_BF16X6) return !(id == 3 || id == 7 || id == 11 || (id >= 15 && id <= 17));
  return true;
}

void mp_config(int id, int* wn, int* wm, int* wc) {
  *wn = kCfgs[id].wn; *wm = kCfgs[id].wm; *wc = kCfgs[id].wc;
}

// Default configuration for a K x K operator: the two-column-group tile whose
// block width covers K most tightly (eight waves per block), else the widest
// single-group tile.  (FP64 and FP32 plans only report it.)
int mp_default_config(int K, int prec) {
  if (prec_int8(prec)) return kOzCfg;
  const int frags = (K + 15) / 16;
  int best = -1, best_cb = 1 << 30;
  for (int id = 0; id < kNumCfgs; ++id) {
    const MpCfg& c = kCfgs[id];
    if (c.wc != 2 || c.wm == 4 || !mp_config_allowed(id, prec)) continue;
    const int cb = c.wn * c.wc;
    if (cb >= frags && cb < best_cb) { best = id; best_cb = cb; }
  }
  if (best >= 0) return best;
  return prec == PREC_F64 ? 13 : 15;   // widest: 256 (FP64) or 512 columns per block
}

constexpr int CHUNK_K = 32;       // k per k-block of the BF16 products
static int split_terms(int prec) { return prec == PREC_BF16X6 ? 3 : 1; }

static void packed_geometry(int K, int* npk, int* nkb) {
  *npk = ((K + 15) / 16) * 16;
  *nkb = (K + CHUNK_K - 1) / CHUNK_K;
}

size_t mp_packed_bytes(int K, int prec) {
  int npk, nkb;
  packed_geometry(K, &npk, &nkb);
  return (size_t)nkb * CHUNK_K * npk * 2 * split_terms(prec);
}

static uint16_t bf16_rne(float f) {
  uint32_t u;
  __builtin_memcpy(&u, &f, 4);
  u += 0x7fffu + ((u >> 16) & 1u);   // round to nearest even
  return (uint16_t)(u >> 16);
}

static double bf16_value(uint16_t h) {
  const uint32_t u = (uint32_t)h << 16;
  float f;
  __builtin_memcpy(&f, &u, 4);
  return (double)f;
}

// Packs B (K x K, row-major, FP64) into the fragment order read by mp_kernel,
// in BF16 (round to nearest even), zero padded.  BF16X6 packs the three BF16 terms of every entry (b = b1 + b2 + b3,
// each the round-to-nearest remainder of the previous, from the FP64 value)
// as three consecutive 16-byte units.
void mp_pack(const double* B, int K, int prec, void* dst) {
  int npk, nkb;
  packed_geometry(K, &npk, &nkb);
  const int CH = 8, T = split_terms(prec);
  uint16_t* o = (uint16_t*)dst;
  const size_t total = (size_t)nkb * CHUNK_K * npk * T;
  for (size_t e = 0; e < total; ++e) o[e] = 0;
  for (int k = 0; k < K; ++k)
    for (int n = 0; n < K; ++n) {
      const int kb = k / CHUNK_K, g = (k % CHUNK_K) / CH, w = k % CH;
      double r = B[(size_t)k * K + n];
      for (int t = 0; t < T; ++t) {
        const uint16_t b = bf16_rne((float)r);
        o[((((size_t)kb * 4 + g) * T + t) * npk + n) * 8 + w] = b;
        r -= bf16_value(b);
      }
    }
}

template <int PREC, class Ti, class To, int WN, int WM, int WC, bool VEC>
static void launch_cfg(const PinvOps& op, int ax, bool fwd, const void* X, void* Y, int rows,
                       int batch, const RhsState* st, int in_scale, int out_scale,
                       const double* la, const double* lb, const double* lc, int a1,
                       const double* gt, hipStream_t s) {
  const int K = op.n[ax];
  const int cb = 16 * WN * WC, ncc = (K + cb - 1) / cb;
  constexpr int BR = WR * 16 * WM;
  const int nrb = (rows + BR - 1) / BR;
  int npk, nkb;
  packed_geometry(K, &npk, &nkb);
  dim3 grid(nrb * ncc, batch);
  hipLaunchKernelGGL((mp_kernel<PREC, Ti, To, WN, WM, WC, VEC>), grid, dim3(64 * WR * WC), 0, s,
                     (const u4*)(fwd ? op.Bf[ax] : op.Bb[ax]), npk, ncc, (const Ti*)X, (To*)Y, K,
                     rows, (int64_t)op.N, st, in_scale, out_scale, la, lb, lc, a1, gt);
}

// Persistent blocks of the operator-resident tile: as many per right-hand
// side as fill the chip once (the operator's LDS share sets the blocks per
// CU), never more than the row tiles.
template <int PREC>
constexpr int res_lds_bytes() {
  return (128 / (4 * MT<PREC>::CH)) * 4 * MT<PREC>::NV * 128 * 16;
}

template <int PREC, class Ti, class To, int WN, int WC>
static void launch_res(const PinvOps& op, int ax, bool fwd, const void* X, void* Y, int rows,
                       int batch, const RhsState* st, int in_scale, int out_scale,
                       const double* la, const double* lb, const double* lc, int a1,
                       const double* gt, hipStream_t s) {
  const int K = op.n[ax];
  constexpr int BR = WR * 16;
  const int nrb = (rows + BR - 1) / BR;
  int npk, nkb;
  packed_geometry(K, &npk, &nkb);
  // LDS per block: the operator, and for BF16 outputs the staged tile
  constexpr int lds_b = res_lds_bytes<PREC>() + (sizeof(To) == 2 ? 128 * (WR * 16 + 8) * 2 : 0);
  constexpr int per_cu = (160 * 1024) / lds_b < 1 ? 1
                         : ((160 * 1024) / lds_b > 4 ? 4 : (160 * 1024) / lds_b);
  const int want = (256 * per_cu + batch - 1) / batch;
  const int nblk = std::max(1, std::min(nrb, want));
  dim3 grid(nblk, batch);
  hipLaunchKernelGGL((mp_res<PREC, Ti, To, WN, WC>), grid, dim3(64 * WR * WC), 0, s,
                     (const u4*)(fwd ? op.Bf[ax] : op.Bb[ax]), npk, (const Ti*)X, (To*)Y, K, rows,
                     (int64_t)op.N, st, in_scale, out_scale, la, lb, lc, a1, gt);
}

template <int PREC, class Ti, class To>
static void launch_mp(int cls, int cfg, const PinvOps& op, int ax, bool fwd, const void* X,
                      void* Y, int batch, const RhsState* st, int in_scale, int out_scale,
                      const double* la, const double* lb, const double* lc, int a1,
                      const double* gt, hipStream_t s, double* rpart = nullptr) {
  trace_begin(cls, s);
  if constexpr (prec_int8(PREC)) {
    (void)cfg;
    launch_oz(op, ax, fwd, X, Y, batch, st, la, lb, lc, a1, gt, rpart, s);
    trace_end(cls, s);
    return;
  } else if constexpr (prec_folds(PREC)) {
    (void)cfg;
    launch_fold(op, ax, fwd, X, sizeof(Ti) == 8, Y, sizeof(To) == 8, batch, st, in_scale,
                out_scale, la, lb, lc, a1, gt, rpart, s);
    trace_end(cls, s);
    return;
  } else {
  const int K = op.n[ax];
  const int rows = (int)(op.N / K);
  const int CH = MT<PREC>::CH;
  if (K % CH != 0) {
    // rows too ragged for 16-byte loads: one scalar-load tile serves every
    // configuration (such grids are small)
    launch_cfg<PREC, Ti, To, 4, 2, 2, false>(op, ax, fwd, X, Y, rows, batch, st, in_scale,
                                             out_scale, la, lb, lc, a1, gt, s);
    trace_end(cls, s);
    return;
  }
#define KP_CASE(ID, W, M_, C)                                                                 \
  case ID:                                                                                    \
    launch_cfg<PREC, Ti, To, W, M_, C, true>(op, ax, fwd, X, Y, rows, batch, st, in_scale,    \
                                             out_scale, la, lb, lc, a1, gt, s);               \
    break;
  if (mp_config_resident(cfg) && K <= 128) {
    if (cfg == kResFirst)
      launch_res<PREC, Ti, To, 8, 1>(op, ax, fwd, X, Y, rows, batch, st, in_scale, out_scale, la,
                                     lb, lc, a1, gt, s);
    else
      launch_res<PREC, Ti, To, 4, 2>(op, ax, fwd, X, Y, rows, batch, st, in_scale, out_scale, la,
                                     lb, lc, a1, gt, s);
    trace_end(cls, s);
    return;
  }
#define KP_COMMON_CASES                                                                      \
  KP_CASE(0, 1, 4, 1) KP_CASE(1, 2, 4, 1) KP_CASE(2, 3, 4, 1) KP_CASE(4, 6, 2, 1)             \
  KP_CASE(5, 8, 2, 1) KP_CASE(6, 12, 1, 1) KP_CASE(8, 2, 4, 2) KP_CASE(9, 3, 4, 2)            \
  KP_CASE(10, 4, 2, 2) KP_CASE(12, 6, 2, 2) KP_CASE(14, 8, 2, 2)                            \
  KP_CASE(18, 8, 1, 1) KP_CASE(19, 4, 1, 2)
  // tiles whose registers would spill are left out: the split's operands are
  // three times as wide, and the FP64-sourced BF16 product holds 16 VGPRs of
  // raw data per row fragment and k-block
  if constexpr (PREC == PREC_BF16) {
    switch (cfg) {
      KP_COMMON_CASES
      KP_CASE(3, 4, 4, 1)
      KP_CASE(7, 16, 1, 1)
      KP_CASE(11, 4, 4, 2)
      KP_CASE(15, 16, 1, 2)
      KP_CASE(17, 8, 4, 2)
      default: KP_CASE(13, 8, 1, 2)
    }
  } else {
    switch (cfg) {
      KP_COMMON_CASES
      default: KP_CASE(13, 8, 1, 2)
    }
  }
#undef KP_COMMON_CASES
#undef KP_CASE
  trace_end(cls, s);
  }
}

// Product q of one application Z = M(R) (Algs. 6-7) for `batch` right-hand
// sides with the solver's buffers: R -> T0 -> T1 -> T0 ... -> Z (R and Z FP64
// in the natural layout, T0 and T1 in the compute type).  The first product
// scales its input per right-hand side and the last unscales its output (not
// in FP64; with op.zf32 the reader of Z does, which finds the product's FP32
// sums in it); the last forward one carries the Hadamard factor, Ghat from the
// eigenvalues or, for the low-rank preconditioner, the table op.gtab.
template <int PREC>
static void pinv_step_t(const PinvOps& op, int q, const double* R, double* Z, void* T0,
                        void* T1, int batch, const RhsState* st, hipStream_t s) {
  using tc = typename MT<PREC>::tc;
  const int scl = (PREC == PREC_F64 || prec_int8(PREC)) ? 0 : 1;
  const int dim = op.dim, ax = q % dim, last = 2 * dim - 1;
  const bool fwd = q < dim;
  void* T[2] = {T0, T1};
  const void* in = q == 0 ? (const void*)R : (const void*)T[(q - 1) % 2];
  void* out = q == last ? (void*)Z : T[q % 2];
  const int cls = fwd ? (ax == 0 ? KC_MP_X_FWD : (ax == 1 ? KC_MP_Y_FWD : KC_MP_Z_FWD))
                      : (ax == 0 ? KC_MP_X_BWD : (ax == 1 ? KC_MP_Y_BWD : KC_MP_Z_BWD));
  if (q == 0) {
    launch_mp<PREC, double, tc>(cls, op.cfg[q], op, ax, fwd, in, out, batch, st, scl, 0, nullptr,
                                nullptr, nullptr, 1, nullptr, s,
                                op.hpart);
  } else if (q == last && op.zf32) {
    if constexpr (PREC != PREC_F64 && !prec_int8(PREC))
      launch_mp<PREC, tc, float>(cls, op.cfg[q], op, ax, fwd, in, out, batch, st, 0, 0, nullptr,
                                 nullptr, nullptr, 1, nullptr, s);
  } else if (q == last) {
    launch_mp<PREC, tc, double>(cls, op.cfg[q], op, ax, fwd, in, out, batch, st, 0, scl, nullptr,
                                nullptr, nullptr, 1, nullptr, s);
  } else if (q == dim - 1 && op.gtab) {
    launch_mp<PREC, tc, tc>(cls, op.cfg[q], op, ax, fwd, in, out, batch, st, 0, 0, nullptr,
                            nullptr, nullptr, 1, op.gtab, s);
  } else if (q == dim - 1) {
    launch_mp<PREC, tc, tc>(cls, op.cfg[q], op, ax, fwd, in, out, batch, st, 0, 0, op.lam[0],
                            dim == 3 ? op.lam[1] : nullptr, op.lam[dim - 1], op.n[0], nullptr, s,
                            op.rpart);
  } else {
    launch_mp<PREC, tc, tc>(cls, op.cfg[q], op, ax, fwd, in, out, batch, st, 0, 0, nullptr,
                            nullptr, nullptr, 1, nullptr, s);
  }
}

template <int PREC>
static void pinv_apply_t(const PinvOps& op, const double* R, double* Z, void* T0, void* T1,
                         int batch, const RhsState* st, hipStream_t s) {
  for (int q = 0; q < 2 * op.dim; ++q) pinv_step_t<PREC>(op, q, R, Z, T0, T1, batch, st, s);
}

// Launches product q of the preconditioner alone (autotuning): q < dim are the
// forward products (the first reads FP64, the last carries G), q >= dim the
// backward ones (the last writes FP64, or FP32 as in a solve: op.zf32).
template <int PREC>
static void product_t(const PinvOps& op, int q, const void* in, void* out, int batch,
                      hipStream_t s) {
  using tc = typename MT<PREC>::tc;
  const int dim = op.dim, ax = q % dim;
  const bool fwd = q < dim;
  const bool gq = q == dim - 1;
  const double* la = gq ? op.lam[0] : nullptr;
  const double* lb = (gq && dim == 3) ? op.lam[1] : nullptr;
  const double* lc = gq ? op.lam[dim - 1] : nullptr;
  const int cls = fwd ? (ax == 0 ? KC_MP_X_FWD : (ax == 1 ? KC_MP_Y_FWD : KC_MP_Z_FWD))
                      : (ax == 0 ? KC_MP_X_BWD : (ax == 1 ? KC_MP_Y_BWD : KC_MP_Z_BWD));
  if (q == 0)
    launch_mp<PREC, double, tc>(cls, op.cfg[q], op, ax, fwd, in, out, batch, nullptr, 0, 0, la,
                                lb, lc, op.n[0], nullptr, s);
  else if (q == 2 * dim - 1 && op.zf32 && !prec_int8(PREC))
    launch_mp<PREC, tc, float>(cls, op.cfg[q], op, ax, fwd, in, out, batch, nullptr, 0, 0, la,
                               lb, lc, op.n[0], nullptr, s);
  else if (q == 2 * dim - 1)
    launch_mp<PREC, tc, double>(cls, op.cfg[q], op, ax, fwd, in, out, batch, nullptr, 0, 0, la,
                                lb, lc, op.n[0], nullptr, s);
  else
    launch_mp<PREC, tc, tc>(cls, op.cfg[q], op, ax, fwd, in, out, batch, nullptr, 0, 0, la, lb,
                            lc, op.n[0], nullptr, s);
}

int pinv_first_blocks(const PinvOps& op) {
  if (prec_int8(op.prec)) return oz_partials(op.N / op.n[0], op.br[0]);
  const int64_t b = op.prec == PREC_F64 ? fold_first_blocks(op) : 0;
  return b > (1 << 30) ? (1 << 30) : (int)b;
}

int pinv_ghat_blocks(const PinvOps& op) {
  if (prec_int8(op.prec)) return oz_partials(op.N / op.n[op.dim - 1], op.br[op.dim - 1]);
  if (prec_folds(op.prec)) {
    const int64_t b = fold_ghat_blocks(op);
    return b > (1 << 30) ? (1 << 30) : (int)b;
  }
  return 0;                   // the BF16 products leave none
}

void pinv_product(const PinvOps& op, int q, const void* in, void* out, int batch,
                  hipStream_t s) {
  switch (op.prec) {
    case PREC_F64: case PREC_F32: break;   // (their tiles follow the size: nothing to choose)
    case PREC_BF16X6: product_t<PREC_BF16X6>(op, q, in, out, batch, s); break;
    case PREC_I8X7: product_t<PREC_I8X7>(op, q, in, out, batch, s); break;
    case PREC_I8X6: product_t<PREC_I8X6>(op, q, in, out, batch, s); break;
    default: product_t<PREC_BF16>(op, q, in, out, batch, s); break;
  }
}

void pinv_step(const PinvOps& op, int q, const double* R, double* Z, void* T0, void* T1,
               int batch, const RhsState* st, hipStream_t s) {
  switch (op.prec) {
    case PREC_F64: pinv_step_t<PREC_F64>(op, q, R, Z, T0, T1, batch, st, s); break;
    case PREC_F32: pinv_step_t<PREC_F32>(op, q, R, Z, T0, T1, batch, st, s); break;
    case PREC_BF16X6: pinv_step_t<PREC_BF16X6>(op, q, R, Z, T0, T1, batch, st, s); break;
    case PREC_I8X7: pinv_step_t<PREC_I8X7>(op, q, R, Z, T0, T1, batch, st, s); break;
    case PREC_I8X6: pinv_step_t<PREC_I8X6>(op, q, R, Z, T0, T1, batch, st, s); break;
    default: pinv_step_t<PREC_BF16>(op, q, R, Z, T0, T1, batch, st, s); break;
  }
}

void pinv_apply(const PinvOps& op, const double* R, double* Z, void* T0, void* T1, int batch,
                const RhsState* st, hipStream_t s) {
  switch (op.prec) {
    case PREC_F64: pinv_apply_t<PREC_F64>(op, R, Z, T0, T1, batch, st, s); break;
    case PREC_F32: pinv_apply_t<PREC_F32>(op, R, Z, T0, T1, batch, st, s); break;
    case PREC_BF16X6: pinv_apply_t<PREC_BF16X6>(op, R, Z, T0, T1, batch, st, s); break;
    case PREC_I8X7: pinv_apply_t<PREC_I8X7>(op, R, Z, T0, T1, batch, st, s); break;
    case PREC_I8X6: pinv_apply_t<PREC_I8X6>(op, R, Z, T0, T1, batch, st, s); break;
    default: pinv_apply_t<PREC_BF16>(op, R, Z, T0, T1, batch, st, s); break;
  }
}

}  // namespace kp
