// FP64 and FP32 mode products of the pseudoinverse (Algs. 6 and 7), folded by
// the symmetry of the eigenvectors.
//
// A product C[r][n] = sum_k X[r][k] B[k][n] contracts the contiguous axis and
// stores Y[n][r] (the rotating layout of kp_modeprod.hip).  The eigenvectors
// of the Dirichlet, Neumann and periodic operators come in G = 2 or 4 groups
// by their parity (kp_basis.cpp, fold_basis), so that with m = ceil(K / G)
//   forward:  X is folded along k into G vectors of m sums and differences,
//             and group q's modes need only the q-th one: G products of
//             m x m instead of one of K x K;
//   backward: the G groups of modes are summed separately over m positions,
//             and the sums are unfolded into the K outputs.
// Both take 1/G of the matrix operations.  G = 1 is the plain product: the
// mixed operators, axes too short to gain, and every FP32 product (whose
// results are those of a plain FP32 sum over k).
//
// A block owns BR = 16 WM WR rows and 16 WN WC positions of every group (four
// waves, WR x WC).  Its rows are loaded in stages of KS k-blocks (16 folded
// positions), folded in registers, and written to LDS in MFMA fragment order,
// double-buffered with one barrier per stage: the fold is done once per
// block.  Each wave streams the operator fragments of its own columns from
// L2 straight into a ring of registers, PD fragments ahead, so nothing waits
// for another wave inside a stage.
//
// What bounds it.  At 512^3 the four quarter products need 0.47 ms of FP64
// matrix time and 0.43 ms of HBM time (2.1 GB at 5 TB/s): 0.73 ms measured
// back to back, 0.80-0.85 in a solve (matrix cores 0.59-0.64 busy), against
// 2.53-2.57 ms for the plain product it replaces (operator staged through LDS,
// rows straight to registers).  Halves: 0.94 ms matrix time, 1.14-1.25 measured
// (1.27-1.36 in a solve, 0.71-0.79 busy).
// Short products are bound by latency: few rows get small tiles, so that every
// CU has some (2D 300 x 200: 35-50 -> 6-10 us; 100 x 75 x 50: 17-22 -> 5-6 us;
// 192 x 192 x 96, D: 53-56 -> 24-25 us).  MFMA: v_mfma_f64_16x16x4 and
// v_mfma_f32_16x16x4 with the operator as the first operand: a lane then
// holds four positions n of one row r, and 16 lanes store 16 consecutive
// rows of Y's row n.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdio>
#include <type_traits>
#include <vector>

#include "kp_common.h"
#include "kp_internal.h"
#include "kp_layout.h"

namespace kp {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

namespace {

template <int PREC> struct FM;
template <> struct FM<PREC_F64> {
  using tc = double; using acc = d4;
  static constexpr int NV = 2;               // 16-byte units per 4 values
  static __device__ __forceinline__ acc mma(double b, double x, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(b, x, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int col(int lane, int v) { return 4 * v + (lane >> 4); }
};
template <> struct FM<PREC_F32> {
  using tc = float; using acc = f4;
  static constexpr int NV = 1;
  static __device__ __forceinline__ acc mma(float b, float x, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(b, x, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int col(int lane, int v) { return 4 * (lane >> 4) + v; }
};

// k-blocks per stage: a stage is one or two 4-value chunks a thread; few rows
// take more, so that a short contraction waits for memory fewer times.
constexpr int stage_blocks(int G, int wn, int br) {
  return br == 16 ? 4 : ((G * wn >= 4 && br >= 64) ? 1 : 2);
}

struct FoldArgs {
  const u4* B;          // packed operator (fold_pack)
  const void* X;
  void* Y;
  int64_t N;
  int K, rows, m, nf, nkb;   // nf column fragments and nkb k-blocks of 16 per group
  int ncc, nrt;         // column chunks, row tiles
  int vec;              // 16-byte loads along k
  const RhsState* st;
  int in_scale, out_scale;
  const double *la, *lb, *lc;
  int a1;
  const double* gt;
  double* rpart;
};

enum FoldMode { FOLD_BWD = 0, FOLD_FWD, FOLD_HAD };

template <class T>
__device__ __forceinline__ void ld4(const T* __restrict__ p, T (&v)[4]) {
  constexpr int U = (int)sizeof(T) / 4;      // 16-byte units of four values
#pragma unroll
  for (int q = 0; q < U; ++q) {
    const u4 u = reinterpret_cast<const u4*>(p)[q];
    __builtin_memcpy(reinterpret_cast<char*>(v) + 16 * q, &u, 16);
  }
}

// The raw values behind folded positions k0 .. k0+3 of one row.  Forward:
// v[0] = x_j, v[1] = x_{K-1-j}, v[2] = x_{h-1-j}, v[3] = x_{h+j} (h = K/2),
// the mirrored ones in ascending memory order (v[1][3-s] belongs to k0+s).
// Backward: v[q] = the q-th group's modes.  Positions past m read valid
// values of the row, masked when folded.
template <class Ti, int G, bool FWD>
__device__ __forceinline__ void fold_load(const Ti* __restrict__ x, int K, int m, int k0,
                                          bool vec, Ti (&v)[G][4]) {
  const int h = K >> 1;
  if (vec) {
    const int k = k0 < m ? k0 : 0;
    ld4(x + k, v[0]);
    if constexpr (FWD) {
      if constexpr (G >= 2) ld4(x + (K - 4 - k), v[1]);
      if constexpr (G == 4) {
        ld4(x + (h - 4 - k), v[2]);
        ld4(x + (h + k), v[3]);
      }
    } else {
#pragma unroll
      for (int q = 1; q < G; ++q) ld4(x + q * m + k, v[q]);
    }
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + s < m ? k0 + s : m - 1;
      v[0][s] = x[k];
      if constexpr (FWD) {
        if constexpr (G >= 2) v[1][3 - s] = x[K - 1 - k];
        if constexpr (G == 4) {
          v[2][3 - s] = x[h - 1 - k];
          v[3][s] = x[h + k];
        }
      } else {
#pragma unroll
        for (int q = 1; q < G; ++q) v[q][s] = x[min(q * m + k, K - 1)];
      }
    }
  }
}

// Folded values f[q][s] of positions k0 + s, rounded once to the compute
// type; 0 past the end.  The centre of an odd axis is its own mirror image.
template <int PREC, class Ti, int G, bool FWD>
__device__ __forceinline__ void fold_vals(const Ti (&v)[G][4], int K, int m, int k0,
                                          double scale, typename FM<PREC>::tc (&f)[G][4]) {
  using tc = typename FM<PREC>::tc;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = k0 + s;
    if constexpr (!FWD || G == 1) {
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const bool in = k < m && q * m + k < K;
        tc t;
        if constexpr (std::is_same<Ti, tc>::value) t = v[q][s];
        else t = (tc)((double)v[q][s] * scale);
        f[q][s] = in ? t : (tc)0;
      }
    } else {
      const bool in = k < m;
      double a = (double)v[0][s], b = (double)v[1][3 - s];
      if constexpr (G == 2) {
        if (2 * k == K - 1) b = 0;
        a *= scale;
        b *= scale;
        f[0][s] = in ? (tc)(a + b) : (tc)0;
        f[1][s] = in ? (tc)(a - b) : (tc)0;
      } else {
        double c = (double)v[2][3 - s], d = (double)v[3][s];
        a *= scale;
        b *= scale;
        c *= scale;
        d *= scale;
        const double s0 = a + b, d0 = a - b, s1 = c + d, d1 = c - d;
        f[0][s] = in ? (tc)(s0 + s1) : (tc)0;
        f[1][s] = in ? (tc)(s0 - s1) : (tc)0;
        f[2][s] = in ? (tc)(d0 + d1) : (tc)0;
        f[3][s] = in ? (tc)(d0 - d1) : (tc)0;
      }
    }
  }
}

// The sum and the sum of squares of a chunk's values, each entry of the row
// once.
template <class Ti, int G>
__device__ __forceinline__ void fold_sums(const Ti (&v)[G][4], int K, int m, int k0,
                                          double (&f)[3]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const int k = k0 + (G == 4 && (q == 1 || q == 2) ? 3 - s : (q == 1 ? 3 - s : s));
      if (k >= m || (G == 2 && q == 1 && 2 * k == K - 1)) continue;   // (the centre, once)
      const double x = (double)v[q][s];
      f[0] += x;
      f[1] += x * x;
    }
  }
}

// rpart: with the Ghat epilogue (lc), the spectral inner products of the block.
// The inputs are then the coefficients rhat of R in the eigenbasis and the
// outputs those of Z = M(R), so by Parseval <R, Z> = sum rhat zhat, ||Z||^2 =
// sum zhat^2 and <L Z, Z> = sum lambda zhat^2 (Z has no component on the null
// space, where Ghat is 0, so its sum is taken as 0).  In a plain forward
// product, the sum and the sum of squares of X's entries.
//
// MODE: backward; a plain forward product; a forward one with the Hadamard
// factor (Ghat or a table) and its sums.  The factor's epilogue, with its
// tests per element, cost plain products up to a fifth of their time (64^3 FP64,
// x: 5.2 -> 4.0 us; 256^3: 74 -> 67; 256 x 256 x 128 FP32, y: 48.6 -> 44.8).
template <int PREC, class Ti, class To, int G, int MODE, int WM, int WN, int WR>
__global__ __launch_bounds__(256, 2) void mp_fold(const FoldArgs a) {
  constexpr bool FWD = MODE != FOLD_BWD, HAD = MODE == FOLD_HAD;
  using M = FM<PREC>;
  using tc = typename M::tc;
  constexpr int NV = M::NV;
  constexpr int WC = 4 / WR;
  constexpr int BR = 16 * WM * WR;                       // rows per block
  constexpr int BRP = BR + 4 / NV;                       // padded (bank-conflict free stores)
  constexpr int KS = stage_blocks(G, WN, BR);            // k-blocks per stage
  constexpr int NTASK = KS * 4 * BR;                     // 4-value chunks per stage
  constexpr int TPT = (NTASK + 255) / 256;
  constexpr int F = KS * G * WN;                         // operator fragments per stage
  constexpr int PD = F < 4 ? F : 4;                      // operator ring depth
  static_assert(F % PD == 0, "ring slots repeat every stage");

  const int rhs = blockIdx.y;
  if (a.st && a.st[rhs].done) return;
  // the column chunks of a row tile run next to each other on one XCD
  int rt, cc;
  if (a.ncc == 1) {
    rt = blockIdx.x;
    cc = 0;
  } else {
    const int grp = blockIdx.x / (8 * a.ncc), rem = blockIdx.x % (8 * a.ncc);
    cc = rem / 8;
    rt = grp * 8 + rem % 8;
    if (rt >= a.nrt) return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / WC, wc = wave % WC;
  const int g = lane >> 4, l16 = lane & 15;
  const int r0 = rt * BR;
  const int K = a.K, m = a.m, rows = a.rows, nkb = a.nkb, nf = a.nf;
  const Ti* X = (const Ti*)a.X + (int64_t)rhs * a.N;
  const bool vec = a.vec != 0;
  const double scale = (a.st && a.in_scale) ? a.st[rhs].scale : 1.0;
  const int jf0 = (cc * WC + wc) * WN;                   // first column fragment
  const bool live = jf0 < nf;
  const bool insum = MODE == FOLD_FWD && a.rpart;
  double fs[3] = {0.0, 0.0, 0.0};

  __shared__ u4 lds[2][KS * G * 4 * NV * BRP];

  // this thread's chunks of a stage: row, k-block within the stage, k group
  const Ti* xrow[TPT];
  int tk[TPT], tat[TPT];
#pragma unroll
  for (int t = 0; t < TPT; ++t) {
    const int id = tid + t * 256;
    const int tg = id & 3, tr = (id >> 2) % BR, tb = (id >> 2) / BR;
    const int r = r0 + tr;
    xrow[t] = X + (int64_t)(r < rows ? r : 0) * K;
    tk[t] = tb * 16 + 4 * tg;
    tat[t] = ((tb * G * 4 + tg) * NV) * BRP + tr;        // group q adds 4 NV BRP q
  }
  constexpr bool EVEN = NTASK % 256 == 0;
  const bool mine = EVEN || tid < NTASK;

#define KP_FOLD_PUT(buf, st_)                                                             \
  if (mine) {                                                                             \
    _Pragma("unroll") for (int t = 0; t < TPT; ++t) {                                     \
      if (insum && r0 + ((tid + t * 256) >> 2) % BR < rows)                               \
        fold_sums<Ti, G>(raw[t], K, m, (st_) * KS * 16 + tk[t], fs);                      \
      tc f[G][4];                                                                         \
      fold_vals<PREC, Ti, G, FWD>(raw[t], K, m, (st_) * KS * 16 + tk[t], scale, f);       \
      _Pragma("unroll") for (int q = 0; q < G; ++q)                                       \
        _Pragma("unroll") for (int h = 0; h < NV; ++h) {                                  \
          u4 u;                                                                           \
          __builtin_memcpy(&u, reinterpret_cast<const char*>(f[q]) + 16 * h, 16);         \
          lds[buf][tat[t] + (q * 4 * NV + h) * BRP] = u;                                  \
        }                                                                                 \
    }                                                                                     \
  }

  // operator fragment f of stage st_: k-block st_ KS + f / (G WN), group, column
  const u4* bp = a.B + lane;
#define KP_FOLD_B(slot, st_, f_)                                                          \
  {                                                                                       \
    const int kk_ = (f_) / (G * WN), q_ = ((f_) / WN) % G, jn_ = (f_) % WN;               \
    const int kb_ = min((st_) * KS + kk_, nkb - 1), jf_ = min(jf0 + jn_, nf - 1);         \
    const u4* s_ = bp + fold_units(fold_block(q_, jf_, kb_, nf, nkb), NV * 64);           \
    _Pragma("unroll") for (int h = 0; h < NV; ++h) breg[slot][h] = s_[h * 64];            \
  }

  typename M::acc acc[G][WM][WN];
#pragma unroll
  for (int q = 0; q < G; ++q)
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[q][i][j][v] = 0;

  Ti raw[TPT][G][4];
  u4 breg[PD][NV];
#pragma unroll
  for (int t = 0; t < TPT; ++t) fold_load<Ti, G, FWD>(xrow[t], K, m, tk[t], vec, raw[t]);
#pragma unroll
  for (int f = 0; f < PD; ++f) KP_FOLD_B(f, 0, f)
  KP_FOLD_PUT(0, 0)
  __syncthreads();

  const int nst = (nkb + KS - 1) / KS;
  for (int s = 0; s < nst; ++s) {
    const int buf = s & 1;
    if (s + 1 < nst) {
#pragma unroll
      for (int t = 0; t < TPT; ++t)
        fold_load<Ti, G, FWD>(xrow[t], K, m, (s + 1) * KS * 16 + tk[t], vec, raw[t]);
    }
    if (live) {
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        const bool on = KS == 1 || s * KS + kk < nkb;
#pragma unroll
        for (int q = 0; q < G; ++q) {
          tc xa[WM][4];
#pragma unroll
          for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int h = 0; h < NV; ++h) {
              const u4 u = lds[buf][(((kk * G + q) * 4 + g) * NV + h) * BRP +
                                    (wr * WM + i) * 16 + l16];
              __builtin_memcpy(reinterpret_cast<char*>(xa[i]) + 16 * h, &u, 16);
            }
#pragma unroll
          for (int j = 0; j < WN; ++j) {
            const int f = (kk * G + q) * WN + j;
            tc b[4];
            __builtin_memcpy(b, breg[f % PD], 16 * NV);
            if (on) {
#pragma unroll
              for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < WM; ++i)
                  acc[q][i][j] = M::mma(b[e], xa[i][e], acc[q][i][j]);
            }
            KP_FOLD_B(f % PD, s, f + PD)
          }
        }
      }
    }
    if (s + 1 < nst) {
      KP_FOLD_PUT(buf ^ 1, s + 1)
      __syncthreads();
    }
  }
#undef KP_FOLD_PUT
#undef KP_FOLD_B

  // ---- epilogue: unfold, Hadamard factor, output scale, transposed store ---
  const double oscale = (a.st && a.out_scale) ? a.st[rhs].inv_scale : 1.0;
  To* Y = (To*)a.Y + (int64_t)rhs * a.N;
  if constexpr (HAD) {
    // The column's eigenvalues (or the rows' table entries) of a fragment are
    // requested while the one before it is computed and stored: a load behind
    // a store to Y waits for nothing but must not be moved ahead of it by the
    // compiler, and one at a time they took longer than the arithmetic (192 x
    // 192 x 96 P: 26.3 -> 23.2 us, 64^3 DN: 5.8 -> 5.0, 256^3 DN: 171 -> 159).
    double rs[WM];
    int rr[WM];
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      const int r = r0 + (wr * WM + i) * 16 + l16;
      rr[i] = r;
      const int rc = min(r, rows - 1);
      rs[i] = a.lc ? a.la[rc % a.a1] + (a.lb ? a.lb[rc / a.a1] : 0.0) : 0.0;
    }
    auto at = [&](int f, int v) {           // mode of element v of fragment f, or -1
      const int q = f / WN, p = (jf0 + f % WN) * 16 + M::col(lane, v), n = q * m + p;
      return p < m && n < K ? n : -1;
    };
    auto factor = [&](int f, double (&w)[WM][4]) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = max(at(f, v), 0);
#pragma unroll
        for (int i = 0; i < WM; ++i)
          if (a.lc) w[i][v] = i == 0 ? a.lc[n] : w[0][v];
          else w[i][v] = a.gt[(int64_t)n * rows + min(rr[i], rows - 1)];
      }
    };
    if (live) {
      double cur[WM][4], nxt[WM][4];
      factor(0, cur);
#pragma unroll
      for (int f = 0; f < G * WN; ++f) {
        if (f + 1 < G * WN) factor(f + 1, nxt);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int n = at(f, v);
#pragma unroll
          for (int i = 0; i < WM; ++i) {
            const double rhat = (double)acc[f / WN][i][f % WN][v];
            const double sum = rs[i] + cur[i][v];
            double val;
            if (!a.lc) val = rhat * cur[i][v];
            else if constexpr (PREC == PREC_F64) val = rhat * ghat_fast(sum);
            else val = fabs(sum) < 1e-13 ? 0.0 : (double)((float)rhat * __frcp_rn((float)sum));
            const To out = (To)val;
            if (n < 0 || rr[i] >= rows) continue;
            if constexpr (PREC == PREC_F64) {   // (used where rpart is set)
              const double z2 = (double)out * (double)out;
              fs[0] += rhat * (double)out;
              fs[1] += z2;
              fs[2] += sum * z2;
            }
            Y[(int64_t)n * rows + rr[i]] = out;
          }
        }
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) cur[i][v] = nxt[i][v];
      }
    }
  } else if (live) {
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      const int r = r0 + (wr * WM + i) * 16 + l16;
      const bool rok = r < rows;
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int p = (jf0 + j) * 16 + M::col(lane, v);   // position within a group
          if (!rok || p >= m) continue;
          if constexpr (FWD) {
#pragma unroll
            for (int q = 0; q < G; ++q) {
              const int n = q * m + p;
              if (G == 2 && n >= K) continue;
              Y[(int64_t)n * rows + r] = (To)acc[q][i][j][v];
            }
          } else {
            double y[4];
            if constexpr (G == 1) {
              y[0] = (double)acc[0][i][j][v];
            } else if constexpr (G == 2) {
              const double e = (double)acc[0][i][j][v], o = (double)acc[1][i][j][v];
              y[0] = e + o;
              y[1] = e - o;
            } else {
              const double e0 = (double)acc[0][i][j][v], e1 = (double)acc[1][i][j][v];
              const double o0 = (double)acc[2][i][j][v], o1 = (double)acc[3][i][j][v];
              const double s0 = e0 + e1, s1 = e0 - e1, t0 = o0 + o1, t1 = o0 - o1;
              y[0] = s0 + t0;
              y[1] = s0 - t0;
              y[2] = s1 + t1;
              y[3] = s1 - t1;
            }
            const int h = K >> 1;
            const int n[4] = {p, K - 1 - p, h - 1 - p, h + p};
#pragma unroll
            for (int q = 0; q < G; ++q) {
              if (G == 2 && q == 1 && n[1] == p) continue;   // the centre of an odd axis
              Y[(int64_t)n[q] * rows + r] = (To)(a.out_scale ? y[q] * oscale : y[q]);
            }
          }
        }
    }
  }
  if (FWD && a.rpart && (HAD ? a.lc != nullptr : cc == 0)) {
    // fixed-order block reduction: lanes, then waves in order
    __shared__ double fred[4][3];
#pragma unroll
    for (int e = 0; e < 3; ++e) fs[e] = wave_sum(fs[e]);
    if (lane == 0) {
#pragma unroll
      for (int e = 0; e < 3; ++e) fred[wave][e] = fs[e];
    }
    __syncthreads();
    if (tid == 0) {
      double t[3] = {0.0, 0.0, 0.0};
      for (int w = 0; w < 4; ++w)
        for (int e = 0; e < 3; ++e) t[e] += fred[w][e];
      if (HAD) {
        const int slot = rt * a.ncc + cc;
        slot_ptr(a.rpart, rhs, S_DOT)[slot] = t[0];
        slot_ptr(a.rpart, rhs, S_SUM)[slot] = 0.0;
        slot_ptr(a.rpart, rhs, S_SQ)[slot] = t[1];
        slot_ptr(a.rpart, rhs, S_AUX2)[slot] = t[2];
      } else {
        slot_ptr(a.rpart, rhs, S_TSUM)[rt] = t[0];
        slot_ptr(a.rpart, rhs, S_TSQ)[rt] = t[1];
      }
    }
  }
}

// Tile shapes: fragments of rows (wm) and, per group, of positions (wn) per
// wave, and row groups of waves (wr).
struct FoldShape { int wm, wn, wr; };

int block_rows(const FoldShape& s) { return 16 * s.wm * s.wr; }
int block_frags(const FoldShape& s) { return s.wn * (4 / s.wr); }

// size class 0 (small), 1, 2 (large) of a G-fold product
FoldShape shape_of(int G, int size, int wr) {
  if (size == 2) return {2, 8 / G, wr};
  if (size == 1) return {2, 4 / G, wr};
  return {1, G == 1 ? 2 : 1, wr};
}

// The shape with the least estimated time (us) for `rows` rows, all right-hand
// sides.  The estimate's terms, each fitted to measured products:
//   matrix  a CU's share of the blocks at its MFMA rate, idle columns
//           included; one-row-fragment waves re-read the operator for every
//           fragment (x 1.15 in FP64, x 1.5 in FP32, whose MFMAs are half as
//           long: 256 x 256 x 128 FP32 58 us against 50)
//   memory  one read per column chunk, the later ones mostly from L2
//           (+ 0.4 each), and one write; 16-row blocks store 128-byte pieces
//           (x 1.4: 16 of 128^3, K = 128, 210 us against 125), 128-row ones
//           leave room for one or two blocks per CU (x 1.2: 64 of 64^3, 60 us
//           against 49)
//   with more than four blocks per CU, one's loads and stores overlap
//   another's matrix work; with fewer they add up, and each stage waits for
//   its loads (0.9 us).
FoldShape choose_shape(int K, int G, int64_t rows, int prec) {
  const bool f64 = prec == PREC_F64;
  const int m = (K + G - 1) / G, nf = (m + 15) / 16;
  const double rate = f64 ? 0.285e6 : 0.57e6;                // flops per us of a CU
  const double bytes = (double)rows * K * (f64 ? 16.0 : 8.0);
  FoldShape best{};
  double least = 0.0;
  for (int size = 0; size < 3; ++size)
    for (int wr = 1; wr <= 4; wr *= 2) {
      if (size == 2 && (wr == 4 || wr * G > 4)) continue;    // not built (registers)
      if (G == 4 && size == 1 && wr == 4) continue;          // not built (LDS)
      const FoldShape s = shape_of(G, size, wr);
      const int bf = block_frags(s), br = block_rows(s);
      const int64_t ncc = (nf + bf - 1) / bf;
      const int64_t per_cu = ((rows + br - 1) / br * ncc + 255) / 256;
      const double mfma = (double)per_cu * br * bf * 16.0 * G * nf * 16.0 * 2.0 / rate *
                          (size == 0 ? (f64 ? 1.15 : 1.5) : 1.0);
      const double mem = bytes * (1.0 + 0.4 * (ncc - 1)) * (br == 16 ? 1.4 : br == 128 ? 1.2 : 1.0) / 5.0e6;
      const int ks = stage_blocks(G, s.wn, br);
      const double t = per_cu <= 4 ? mfma + mem + 0.9 * ((nf + ks - 1) / ks)
                                   : std::max(mfma, mem) + 0.3 * std::min(mfma, mem);
      if (least == 0.0 || t < least) {
        least = t;
        best = s;
      }
    }
  return best;
}

// Column chunks, row tiles and blocks per right-hand side of a product over K
// points in G groups (the tiles of several chunks go in rounds of eight, one
// per XCD).
struct FoldGrid { int nf, ncc, nrt, blocks; };
FoldGrid grid_of(int K, int G, int rows, const FoldShape& s) {
  FoldGrid g;
  g.nf = ((K + G - 1) / G + 15) / 16;
  g.ncc = (g.nf + block_frags(s) - 1) / block_frags(s);
  g.nrt = (rows + block_rows(s) - 1) / block_rows(s);
  g.blocks = (g.ncc == 1 ? g.nrt : (g.nrt + 7) / 8 * 8) * g.ncc;
  return g;
}

template <int PREC, class Ti, class To, int G, int MODE>
void launch_shape(const FoldShape& s, const FoldArgs& a, int blocks, int batch, hipStream_t st) {
  const dim3 grid(blocks, batch), blk(256);
#define KP_F(WM, WN, WR)                                                                    \
  if (s.wm == WM && s.wn == WN && s.wr == WR) {                                             \
    hipLaunchKernelGGL((mp_fold<PREC, Ti, To, G, MODE, WM, WN, WR>), grid, blk, 0, st, a);   \
    return;                                                                                 \
  }
  KP_F(2, 8 / G, 1)
  if constexpr (G != 4) { KP_F(2, 8 / G, 2) }
  KP_F(2, 4 / G, 1) KP_F(2, 4 / G, 2)
  if constexpr (G != 4) { KP_F(2, 4 / G, 4) }
  constexpr int WS = G == 1 ? 2 : 1;
  KP_F(1, WS, 1) KP_F(1, WS, 2) KP_F(1, WS, 4)
#undef KP_F
}

template <int PREC, class Ti, class To>
void launch_types(int G, int mode, const FoldShape& s, const FoldArgs& a, int blocks, int batch,
                  hipStream_t st) {
  if constexpr (PREC == PREC_F64) {
#define KP_G(G_)                                                                            \
  if (G == G_) {                                                                            \
    if (mode == FOLD_FWD)                                                                   \
      return launch_shape<PREC, Ti, To, G_, FOLD_FWD>(s, a, blocks, batch, st);             \
    if (mode == FOLD_HAD)                                                                   \
      return launch_shape<PREC, Ti, To, G_, FOLD_HAD>(s, a, blocks, batch, st);             \
    return launch_shape<PREC, Ti, To, G_, FOLD_BWD>(s, a, blocks, batch, st);               \
  }
    KP_G(4) KP_G(2) KP_G(1)
#undef KP_G
  } else {
    // FP32: unfolded, so a plain forward product is a backward one with the
    // other operator; only the first product reads FP64 and only the last one
    // writes it, and neither carries the factor (a 2D plan's second one does)
    if constexpr (std::is_same<Ti, float>::value && std::is_same<To, float>::value)
      if (mode == FOLD_HAD)
        return launch_shape<PREC, Ti, To, 1, FOLD_HAD>(s, a, blocks, batch, st);
    launch_shape<PREC, Ti, To, 1, FOLD_BWD>(s, a, blocks, batch, st);
  }
}

}  // namespace

// Partial sums per right-hand side of the product along the last axis (a
// function of the grid only).
int64_t fold_ghat_blocks(const PinvOps& op) {
  const int ax = op.dim - 1, K = op.n[ax], G = op.fold[ax];
  const FoldGrid g = grid_of(K, G, (int)(op.N / K), choose_shape(K, G, op.N / K, op.prec));
  return (int64_t)g.nrt * g.ncc;
}

// Row tiles of the first product (the partial sums of its input).
int64_t fold_first_blocks(const PinvOps& op) {
  const int K = op.n[0], G = op.fold[0];
  return grid_of(K, G, (int)(op.N / K), choose_shape(K, G, op.N / K, op.prec)).nrt;
}

// Product q's kernel, as its template's name and total threads (a solve's, with
// the partial sums it leaves, chooses by one right-hand side's rows).
void fold_kernel_name(const PinvOps& op, int q, int batch, char* name, size_t len) {
  const int dim = op.dim, ax = q % dim, K = op.n[ax], G = op.fold[ax], rows = (int)(op.N / K);
  const bool f64 = op.prec == PREC_F64, had = q == dim - 1;
  const FoldShape s = choose_shape(K, G, had ? rows : (int64_t)rows * batch, op.prec);
  const int mode = had ? FOLD_HAD : (f64 && q < dim ? FOLD_FWD : FOLD_BWD);
  snprintf(name, len, "kp::mp_fold<%d, %s, %s, %d, %d, %d, %d, %d>|%lld", op.prec,
           f64 || q == 0 ? "double" : "float",
           f64 || (q == 2 * dim - 1 && !op.zf32) ? "double" : "float", G, mode, s.wm, s.wn, s.wr,
           256LL * grid_of(K, G, rows, s).blocks * batch);
}

void launch_fold(const PinvOps& op, int ax, bool fwd, const void* X, bool in_f64, void* Y,
                 bool out_f64, int batch, const RhsState* st, int in_scale, int out_scale,
                 const double* la, const double* lb, const double* lc, int a1, const double* gt,
                 double* rpart, hipStream_t s) {
  const int K = op.n[ax], G = op.fold[ax];
  const int rows = (int)(op.N / K);
  FoldArgs a{};
  a.B = (const u4*)(fwd ? op.Bf[ax] : op.Bb[ax]);
  a.X = X;
  a.Y = Y;
  a.N = op.N;
  a.K = K;
  a.rows = rows;
  a.m = (K + G - 1) / G;
  // partial sums may not depend on the batch
  const FoldShape sh = choose_shape(K, G, lc || rpart ? rows : (int64_t)rows * batch, op.prec);
  const FoldGrid g = grid_of(K, G, rows, sh);
  a.nf = a.nkb = g.nf;
  a.ncc = g.ncc;
  a.nrt = g.nrt;
  // 16-byte loads of four consecutive values need every segment's start at a
  // multiple of 16 bytes and, backward, groups that end on a whole chunk
  const int al = in_f64 ? 2 : 4;
  if (fwd) {
    if (G == 1) a.vec = K % 4 == 0;
    else if (G == 2) a.vec = K % al == 0 && K >= 8;
    else a.vec = K % (2 * al) == 0;
  } else {
    a.vec = K % (4 * G) == 0;
  }
  a.st = st;
  a.in_scale = in_scale;
  a.out_scale = out_scale;
  a.la = la;
  a.lb = lb;
  a.lc = lc;
  a.a1 = a1;
  a.gt = gt;
  a.rpart = rpart;
  const int mode = !fwd ? FOLD_BWD : ((lc || gt) ? FOLD_HAD : FOLD_FWD);
  if (op.prec == PREC_F64) launch_types<PREC_F64, double, double>(G, mode, sh, a, g.blocks, batch, s);
  else if (in_f64) launch_types<PREC_F32, double, float>(G, mode, sh, a, g.blocks, batch, s);
  else if (out_f64) launch_types<PREC_F32, float, double>(G, mode, sh, a, g.blocks, batch, s);
  else launch_types<PREC_F32, float, float>(G, mode, sh, a, g.blocks, batch, s);
}

size_t fold_packed_bytes(int K, int G, int prec) {
  const size_t p = (size_t)(((K + G - 1) / G + 15) / 16) * 16;
  return G * p * p * (prec == PREC_F64 ? 8 : 4);
}

// Packs the folded basis Qh (fold_basis: m x K, group-ordered columns) for
// the forward product (k = position, n = mode of the group) or the backward
// one (k = mode, n = position).  16-byte unit (q, jf, kb, h, lane) at
// (((q nf + jf) nkb + kb) NV + h) 64 + lane; lane 16 g + c holds
// k = 16 kb + 4 g .. + 3 of column 16 jf + c (FP64: two of them per unit h).
void fold_pack(const double* Qh, int K, int G, bool fwd, int prec, void* dst) {
  const int m = (K + G - 1) / G, nb = (m + 15) / 16;
  const int NV = prec == PREC_F64 ? 2 : 1, per = 4 / NV;
  // (dst is zeroed: only existing entries are written)
  for (int q = 0; q < G; ++q) {
    const int cnt = std::min(m, K - q * m);
    for (int pos = 0; pos < m; ++pos)
      for (int mode = 0; mode < cnt; ++mode) {
        const int k = fwd ? pos : mode, n = fwd ? mode : pos;
        const double v = Qh[(size_t)pos * K + q * m + mode];
        const size_t unit = fold_units(fold_block(q, n / 16, k / 16, nb, nb), NV) + (k % 4) / per;
        const size_t at = (unit * 64 + 16 * ((k % 16) / 4) + n % 16) * per + k % per;
        if (prec == PREC_F64) ((double*)dst)[at] = v;
        else ((float*)dst)[at] = (float)v;
      }
  }
}

}  // namespace kp
