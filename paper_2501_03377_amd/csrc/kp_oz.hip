// FP64-accurate mode products on the int8 matrix cores (PREC_I8X7, PREC_I8X6),
// after the splitting idea of Ozaki et al.: every value is a short sum of
// small integers times powers of two, the integer products are exact on the
// matrix cores, and only their recombination rounds.  S digits per value:
//   S = 7 (I8X7).  A row of values along the contracted axis gets the power of
//   two 2^e with |x| < 2^e and is cut into 7 digits,
//       x = 2^e sum_i a_i 128^-(i+1),  a_i integers in [-127, 127]
//   (truncation at every step, so all digits carry the sign of x and a
//   small value has small digits; the remainder after the seventh is below
//   2^(e - 49)).  Digits of one sign matter here: with two's complement
//   digits a small negative value has large low digits, and the dropped
//   products below would then carry the full 2^-49 scale for every such
//   value.
//   S = 6 (I8X6).  2^e with |x| < 2^e * 126/128, the image
//   F = trunc(x 2^(47 - e)) (|F| < 126 * 2^40) and its balanced base-256
//   digits, low to high with carries,
//       F = sum_i d_i 256^(5-i),  d_i in [-128, 127], |d_0| <= 126,
//   so x = 2^(e - 47) sum_i d_i 256^(5-i) up to the truncation (below
//   2^(e - 47)).  A small value still has small digits (its high digits
//   are zero), and the digits below a cut take either sign, so the dropped
//   products cancel rather than add.
//   Operator: column n of B likewise with 2^f_n, packed at plan time.
//   Product: the digit products with i + j < S are summed exactly in int32
//   by v_mfma_i32_16x16x64_i8, one accumulator per diagonal d = i + j
//   (|sum| <= 7 * 128^2 * K < 2^31 for K <= 512), and recombined in FP64,
//       y = 2^(e + f_n - 14) sum_d base^-d acc_d,  base 128 or 256
//   (for S = 6 the two 2^-47 and the 256^10 of the top diagonal give the
//   same 2^-14).  The error per output is a few units of 2^-49 (S = 7) or
//   2^-48 (S = 6) K max|x_r| max|b_n| at worst, far below what FP64
//   preconditioning needs (one CG iteration).
//
// The products are folded by the eigenvectors' parity as the FP64 ones are
// (kp_fold.hip): G groups of m = K/G sums and differences, each group a row
// of values of its own with its own exponent.
//
// A persistent block sweeps tiles of 32 rows (128 on the shortest axes).  Its
// threads hold the tile's rows (TPR threads a row, PP pairs of positions per thread and group, pair
// c TPR + t to thread t, so that every load covers whole 128-byte lines),
// fold them, find each row's exponents by shuffles and write the digits to
// LDS in the MFMA operand's order: a thread's 2 PP values of a group are
// consecutive k slots, and the operator is packed in that order of k.  Then
// each wave multiplies its own column fragments, the two 16-row fragments
// together, with the operator's digits streamed from L2 into registers: a
// digit's register is refilled with a later k-block's as soon as its last
// product has been issued.  No wave waits for another while it multiplies.
//
// What bounds it.  A 512^3 product moves 2.1 GB, 0.43 ms at 5 TB/s; its matrix
// work is 0.16 ms in four groups and 0.33 ms in two, at the 2.1 GHz the cores
// keep under it.  Measured back to back, S = 6: 0.59-0.60 ms (four), 0.77-0.86
// (two), 1.24-1.25 (one), against 1.30-1.40 for the unfolded kernel it replaces
// (operator digits through LDS a column fragment at a time, the k range split
// over two waves); S = 7: 0.70-0.77 and 0.99-1.05 against 1.59-1.68.  K > 256
// has one block per CU, and a tile's phases add up in it: with the row loads
// left out 0.64 of 0.73 ms remained, without loads and stores 0.44 ms, without
// the digits 0.67 ms, without the recombination 0.70 ms.  Registers bound the
// backward four-group kernel there (12-16 bytes of scratch a lane for S = 6,
// 64-72 for S = 7).  K <= 256 has two blocks per CU, one's phases beside the
// other's: 64 of 128^3 (two groups) 0.46-0.56 ms, 3.8-4.7 TB/s.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdio>
#include <vector>

#include "kp_common.h"
#include "kp_internal.h"

namespace kp {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

namespace {

constexpr int OZ_SMAX = 7;            // most digits per value
constexpr int OZ_BAD = 0x40000000;    // exponent marker of a row with a non-finite value

// The geometry of a product over K points in G groups with tiles of br rows:
// threads per block, threads per row, pairs per thread and group, k-blocks of
// 64 slots and column fragments per group.
struct OzGeom { int nt, br, tpr, pp, nkb, nf; };
OzGeom oz_geom(int K, int G, int br) {
  OzGeom g;
  g.nt = K > 256 ? 512 : 256;
  g.br = br;
  g.tpr = g.nt / br;
  const int m = K / G, need = (m / 2 + g.tpr - 1) / g.tpr;
  g.pp = 16 / G;
  for (int ppg = 4; ppg <= 16; ppg += 4)     // the compiled ones: PP G = 4, 8, 12, 16
    if (ppg / G >= need) { g.pp = ppg / G; break; }
  if (g.nt == 512 && g.pp * G < 12) g.pp = 12 / G;
  g.nkb = (g.tpr * 2 * g.pp + 63) / 64;
  g.nf = (m + 15) / 16;
  return g;
}

// The row's exponent e from its largest magnitude: |x| < 2^e (S = 7), and
// |x| < 2^e * 126/128 for the balanced split (S = 6), whose top digit must
// stay below 127 after the carries.
template <int S>
__device__ __forceinline__ int oz_exponent(double mx) {
  int e = 0;
  if (mx > 0.0) {
    const double m = frexp(mx, &e);
    if (S == 6 && m >= 0.984375) ++e;
  }
  return max(e, -1021);                         // images of subnormal rows fit too
}

// The right shift of the 53-bit significand that gives a value's image,
// plus the biased exponent field: 49 - e bits (S = 7) or 47 - e (S = 6)
// below the binary point.
template <int S>
__device__ __forceinline__ int oz_cshift(int e) { return e + (S == 7 ? 1026 : 1028); }

// Digits of four values, digit s of the four in the bytes of dg[s].
//
// S = 7: the image F = floor(|x| 2^(49 - e)) < 2^49 is the 53-bit significand
// shifted right by e + 1026 - max(ef, 1) >= 4 (ef the biased exponent field;
// cshift = e + 1026, or past 63 for a non-finite row, which shifts everything
// out); its 7-bit fields from the top are the digit magnitudes, which take the
// sign of x (negated two values at a time on 16-bit halves).  These are the
// digits of truncating |x| 2^-e one base-128 place at a time.
//
// S = 6: from the same kind of image, F = floor(|x| 2^(47 - e)) (the
// significand shifted right by cshift - max(ef, 1) >= 6), signed.  Adding 128
// to each of its five low bytes in one 64-bit add, G = F + 0x8080808080, turns
// every low digit d into the byte d + 128 (the digits in [-128, 127] of an
// integer are unique, and d + 128 is its byte of G), so XOR 0x80 gives the
// two's complement digit, four at a time; the top digit is G >> 40
// (arithmetic), at most 126 in magnitude.  A 4 x 4 byte transpose (v_perm_b32)
// then gathers digit s of the four values.
template <int S>
__device__ __forceinline__ void oz_digits(const double (&x)[4], int cshift, unsigned (&dg)[S]) {
  unsigned u[S][4], sg[4], lo[4], hi4[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint64_t bits = (uint64_t)__double_as_longlong(x[c]);
    const unsigned hi = (unsigned)(bits >> 32);
    const unsigned ef = (hi >> 20) & 0x7ffu;
    const unsigned sh = (unsigned)min(cshift - (int)max(ef, 1u), 63);
    const uint64_t sig = ((uint64_t)((hi & 0xfffffu) | (min(ef, 1u) << 20)) << 32) |
                         (bits & 0xffffffffull);
    const uint64_t F = sig >> sh;
    if constexpr (S == 7) {
      const unsigned fh = (unsigned)(F >> 32), fl = (unsigned)F;
      sg[c] = (unsigned)((int)hi >> 31);        // 0 or all ones
      u[0][c] = fh >> 10;
      u[1][c] = (fh >> 3) & 127u;
      u[2][c] = ((fh << 4) | (fl >> 28)) & 127u;
      u[3][c] = (fl >> 21) & 127u;
      u[4][c] = (fl >> 14) & 127u;
      u[5][c] = (fl >> 7) & 127u;
      u[6][c] = fl & 127u;
    } else {
      const uint64_t m = (uint64_t)(int64_t)((int)hi >> 31);   // 0 or all ones
      const uint64_t Gd = ((F ^ m) - m) + 0x8080808080ull;
      lo[c] = (unsigned)Gd ^ 0x80808080u;       // digits 5, 4, 3, 2 (bytes 0..3)
      hi4[c] = (unsigned)(Gd >> 32);            // byte 0: digit 1 + 128, byte 1: digit 0
    }
  }
  if constexpr (S == 7) {
    const unsigned m01 = (sg[0] & 0xffffu) | (sg[1] & 0xffff0000u);
    const unsigned m23 = (sg[2] & 0xffffu) | (sg[3] & 0xffff0000u);
#pragma unroll
    for (int s = 0; s < 7; ++s) {
      // (d ^ m) - m on each 16-bit half negates where m is all ones; the
      // low bytes of the four signed digits then make one dword
      const u16x2 p01 = __builtin_bit_cast(u16x2, (u[s][0] | (u[s][1] << 16)) ^ m01) -
                        __builtin_bit_cast(u16x2, m01);
      const u16x2 p23 = __builtin_bit_cast(u16x2, (u[s][2] | (u[s][3] << 16)) ^ m23) -
                        __builtin_bit_cast(u16x2, m23);
      dg[s] = __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, p23),
                                    __builtin_bit_cast(unsigned, p01), 0x06040200u);
    }
  } else {
    // byte k of value c -> byte c of dword k (two rounds of byte pairs)
    const unsigned l01a = __builtin_amdgcn_perm(lo[1], lo[0], 0x05010400u);
    const unsigned l01b = __builtin_amdgcn_perm(lo[1], lo[0], 0x07030602u);
    const unsigned l23a = __builtin_amdgcn_perm(lo[3], lo[2], 0x05010400u);
    const unsigned l23b = __builtin_amdgcn_perm(lo[3], lo[2], 0x07030602u);
    dg[5] = __builtin_amdgcn_perm(l23a, l01a, 0x05040100u);
    dg[4] = __builtin_amdgcn_perm(l23a, l01a, 0x07060302u);
    dg[3] = __builtin_amdgcn_perm(l23b, l01b, 0x05040100u);
    dg[2] = __builtin_amdgcn_perm(l23b, l01b, 0x07060302u);
    const unsigned h01 = __builtin_amdgcn_perm(hi4[1], hi4[0], 0x05010400u);
    const unsigned h23 = __builtin_amdgcn_perm(hi4[3], hi4[2], 0x05010400u);
    dg[1] = __builtin_amdgcn_perm(h23, h01, 0x05040100u) ^ 0x80808080u;
    dg[0] = __builtin_amdgcn_perm(h23, h01, 0x07060302u);
  }
}

// One output from its exact diagonal sums a[d]: sum_d base^-d a[d] (Horner,
// low diagonals first; base 128 for S = 7, 256 for S = 6), scaled by
// 2^(e + f - 14); NaN for a non-finite row.
template <int S>
__device__ __forceinline__ double oz_value(const int (&a)[S], int e, int f) {
  constexpr double inv = S == 7 ? 1.0 / 128.0 : 1.0 / 256.0;
  double val = (double)a[S - 1];
#pragma unroll
  for (int d = S - 2; d >= 0; --d) val = (double)a[d] + val * inv;
  return e == OZ_BAD ? NAN : ldexp(val, e + f - 14);
}

struct OzArgs {
  const u4* B;          // operator digits (oz_pack)
  const int* fexp;      // exponents of the K columns, in output order of the groups
  const double* X;
  double* Y;
  int64_t N;
  int K, rows, m, nkb, nf, ntiles;
  const RhsState* st;
  const double *la, *lb, *lc;
  int a1;
  const double* gt;
  double* rpart;
};

// The raw values behind a thread's pairs: v[q][c] holds, forward, the pair
// (x_j, x_j+1) (q = 0), its mirror image in memory order (1), and with G = 4
// the pairs mirrored about and shifted by h = K/2 (2, 3); backward, the q-th
// group's modes.  Pairs past m read the row's first ones, zeroed when folded.
template <int G, bool FWD, int PP, int TPR>
__device__ __forceinline__ void oz_load(const double* __restrict__ x, int K, int m, int t,
                                        d2 (&v)[G][PP]) {
  const int h = K >> 1;
#pragma unroll
  for (int c = 0; c < PP; ++c) {
    int j = 2 * (c * TPR + t);
    j = j < m ? j : 0;
    v[0][c] = *reinterpret_cast<const d2*>(x + j);
    if constexpr (FWD) {
      if constexpr (G >= 2) v[1][c] = *reinterpret_cast<const d2*>(x + (K - 2 - j));
      if constexpr (G == 4) {
        v[2][c] = *reinterpret_cast<const d2*>(x + (h - 2 - j));
        v[3][c] = *reinterpret_cast<const d2*>(x + (h + j));
      }
    } else {
#pragma unroll
      for (int q = 1; q < G; ++q) v[q][c] = *reinterpret_cast<const d2*>(x + (q * m + j));
    }
  }
}

// In place: the folded values (0 past m), v[q][c] then the pair of group q.
template <int G, bool FWD, int PP, int TPR>
__device__ __forceinline__ void oz_fold(int m, int t, d2 (&v)[G][PP]) {
#pragma unroll
  for (int c = 0; c < PP; ++c) {
    const bool in = 2 * (c * TPR + t) < m;
    if constexpr (FWD && G == 2) {
      const d2 a = v[0][c], b = {v[1][c].y, v[1][c].x};
      v[0][c] = a + b;
      v[1][c] = a - b;
    } else if constexpr (FWD && G == 4) {
      const d2 a = v[0][c], b = {v[1][c].y, v[1][c].x}, cc = {v[2][c].y, v[2][c].x}, d = v[3][c];
      const d2 s0 = a + b, d0 = a - b, s1 = cc + d, d1 = cc - d;
      v[0][c] = s0 + s1;
      v[1][c] = s0 - s1;
      v[2][c] = d0 + d1;
      v[3][c] = d0 - d1;
    }
#pragma unroll
    for (int q = 0; q < G; ++q)
      if (!in) v[q][c] = (d2){0.0, 0.0};
  }
}

// the value of the neighbouring lane (lane ^ 1), by DPP quad_perm [1, 0, 3, 2]
__device__ __forceinline__ double swap_pair(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0xb1, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0xb1, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// waits for this wave's LDS accesses, not for its global ones
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// rpart: with Ghat (lc), the spectral <R, Z>, ||Z||^2 and <L Z, Z>; in a plain
// forward product, the sum and the sum of squares of X's entries (a
// nonsingular right-hand side's ||eta||^2 when the product is the solve's
// first and X is eta).  One partial per tile.
template <int S, int G, bool FWD, int PP, int NT, int BR>
__global__ __launch_bounds__(NT, 2) void mp_oz(const OzArgs a) {
  constexpr int NW = NT / 64, TPR = NT / BR;
  constexpr int RP = BR / 32;                             // row pairs (of 16-row fragments)
  constexpr int NKB = (TPR * 2 * PP + 63) / 64;           // k-blocks per group
  constexpr int KP = NKB * 64;                            // k slots per group
  constexpr int VAL = 2 * PP;                             // slots per thread and group
  constexpr int DP = BR * 64;                             // bytes of a digit plane
  // digit s of group q, k-block kb, row r: 64 bytes at ((q NKB + kb) S + s) DP + 64 r
  __shared__ u4 dig[G * NKB * S * (DP / 16)];
  __shared__ int sex[G][BR];                              // row exponents of the groups
  __shared__ double srs[BR];                              // eigenvalue sums of the rows (Ghat)
  __shared__ double red[NW][3];
  __shared__ alignas(16) int sfx[512];                    // column exponents and eigenvalues
  __shared__ alignas(32) double slc[FWD ? 512 : 4];

  const int rhs = blockIdx.y;
  if (a.st && a.st[rhs].done) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (scalar: operator addresses are)
  const int g = lane >> 4, l16 = lane & 15;
  const int K = a.K, m = a.m, rows = a.rows, nf = a.nf;
  const int trow = tid / TPR, tt = tid % TPR;             // this thread's row and share of it
  const double* X = a.X + (int64_t)rhs * a.N;
  double* Y = a.Y + (int64_t)rhs * a.N;
  const bool ghat = FWD && a.lc != nullptr;
  const bool insum = FWD && a.rpart && !a.lc && !a.gt;
  for (int i = tid; i < K; i += NT) {
    sfx[i] = a.fexp[i];
    if constexpr (FWD) {
      if (ghat) slc[i] = a.lc[i];
    }
  }
  // slots past the threads' (a short axis) stay zero
  if constexpr (TPR * VAL < KP) {
    for (int i = tid; i < (int)(sizeof(dig) / 16); i += NT) dig[i] = (u4){0, 0, 0, 0};
    __syncthreads();
  }
  // The operator digits of step f (group f / NKB, k-block f % NKB) of column
  // fragment jf; steps past the fragment's are those of fragment jnext.  RD
  // steps are in registers or on their way: a digit's register takes that of
  // RD steps on as soon as its last product is issued.
  constexpr int STEPS = G * NKB;
  // (two where they fit the registers: 2-6% at 512^3)
  constexpr int RD = STEPS % 2 == 0 && S == 6 && (FWD || G < 4 || NT == 256) ? 2 : 1;
  auto bstep = [&](int jf, int f, int jnext) {
    const int j = f < STEPS ? jf : jnext, e = f < STEPS ? f : f - STEPS;
    return a.B + (uint32_t)((((e / NKB) * nf + j) * NKB + e % NKB) * S * 64);
  };

  d2 raw[G][PP];
  auto row_src = [&](int tile) {
    const int r = tile * BR + trow;
    return X + (uint32_t)(((tile < a.ntiles && r < rows) ? r : 0) * K);
  };
  oz_load<G, FWD, PP, TPR>(row_src(blockIdx.x), K, m, tt, raw);
  u4 b[RD][S];
#pragma unroll
  for (int d = 0; d < RD; ++d) {
    const u4* src = bstep(min(wave / RP, nf - 1), d, min((wave + NW) / RP, nf - 1));
#pragma unroll
    for (int s = 0; s < S; ++s) b[d][s] = src[s * 64 + lane];
  }

  for (int tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x) {
    const int r0 = tile * BR;
    double fs0 = 0.0, fs1 = 0.0, fs2 = 0.0;
    if (insum && r0 + trow < rows) {
      // the same values once each: pairs inside m only
#pragma unroll
      for (int c = 0; c < PP; ++c) {
        if (2 * (c * TPR + tt) >= m) continue;
#pragma unroll
        for (int q = 0; q < G; ++q) {
          fs0 += raw[q][c].x + raw[q][c].y;
          fs1 += raw[q][c].x * raw[q][c].x + raw[q][c].y * raw[q][c].y;
        }
      }
    }
    oz_fold<G, FWD, PP, TPR>(m, tt, raw);
#pragma unroll
    for (int q = 0; q < G; ++q) {
      double mx = 0.0;
      int bad = 0;
#pragma unroll
      for (int c = 0; c < PP; ++c) {
        const double x = fabs(raw[q][c].x), y = fabs(raw[q][c].y);
        bad |= !(x <= DBL_MAX) | !(y <= DBL_MAX);
        mx = fmax(mx, fmax(x, y));
      }
#pragma unroll
      for (int o = 1; o < TPR; o <<= 1) {
        mx = fmax(mx, __shfl_xor(mx, o, 64));
        bad |= __shfl_xor(bad, o, 64);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int e = oz_exponent<S>(mx);
      if (tt == 0) sex[q][trow] = bad ? OZ_BAD : e;
      const int cs = bad ? 4096 : oz_cshift<S>(e);
      unsigned char* base = reinterpret_cast<unsigned char*>(dig);
      // four values a round (two pairs), or the last pair alone
      unsigned dw[S][(VAL + 3) / 4];
#pragma unroll
      for (int w = 0; w < (VAL + 3) / 4; ++w) {
        const d2 p0 = raw[q][2 * w];
        const d2 p1 = 2 * w + 1 < PP ? raw[q][2 * w + 1 < PP ? 2 * w + 1 : 0] : (d2){0.0, 0.0};
        const double x4[4] = {p0.x, p0.y, p1.x, p1.y};
        unsigned dg[S];
        oz_digits<S>(x4, cs, dg);
#pragma unroll
        for (int s = 0; s < S; ++s) dw[s][w] = dg[s];
        __builtin_amdgcn_sched_barrier(0);
      }
      // to LDS in the largest pieces that stay inside a 16-byte operand unit
      constexpr int PC = VAL % 16 == 0 ? 16 : (VAL % 8 == 0 ? 8 : (VAL % 4 == 0 ? 4 : 2));
#pragma unroll
      for (int p = 0; p < VAL / PC; ++p) {
        const int slot = tt * VAL + p * PC;
        unsigned char* at = base + (size_t)(q * NKB + slot / 64) * S * DP + trow * 64 + slot % 64;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          unsigned char* o = at + s * DP;
          if constexpr (PC == 16)
            *reinterpret_cast<u4*>(o) =
                (u4){dw[s][4 * p], dw[s][4 * p + 1], dw[s][4 * p + 2], dw[s][4 * p + 3]};
          else if constexpr (PC == 8)
            *reinterpret_cast<uint2*>(o) = make_uint2(dw[s][2 * p], dw[s][2 * p + 1]);
          else if constexpr (PC == 4)
            *reinterpret_cast<unsigned*>(o) = dw[s][p];
          else
            *reinterpret_cast<unsigned short*>(o) =
                (unsigned short)(p & 1 ? dw[s][p / 2] >> 16 : dw[s][p / 2]);
        }
      }
    }
    if (ghat && tid < BR) {
      const int r = min(r0 + tid, rows - 1);
      srs[tid] = a.la[r % a.a1] + (a.lb ? a.lb[r / a.a1] : 0.0);
    }
    lds_barrier();

    const int tnext = tile + gridDim.x;
    // jobs: a column fragment of one row pair; the waves at the same fragment
    // read the same operator digits
    const int jobs = nf * RP;
    for (int job = wave; job < jobs; job += NW) {
      const int jf = job / RP, pr = job % RP;
      const bool last = job + NW >= jobs;
      const int jnext = (last ? wave : job + NW) / RP;
      const int rp = r0 + pr * 32;                        // the pair's first row
      // Outputs x0 and x1 of rows l16 and 16 + l16 at Y's row n: neighbouring
      // lanes trade so that each stores two consecutive rows, 16 bytes (even
      // lanes of the first 16 rows, odd lanes of the others), and one store
      // covers whole 128-byte lines.
      const bool odd = (lane & 1) != 0;
      const int srow = rp + (odd ? 15 : 0) + l16;           // 16 + l16 - 1 for an odd lane
      const bool sok = rp + (odd ? 16 : 0) < rows;
      auto store = [&](double x0, double x1, int n, bool ok) {
        const double give = odd ? x0 : x1, keep1 = odd ? x1 : x0;
        const double got = swap_pair(give);
        if (ok && sok)
          *reinterpret_cast<d2*>(Y + (uint32_t)(n * rows + srow)) =
              odd ? (d2){got, keep1} : (d2){keep1, got};
      };
      const int p = jf * 16 + 4 * g;                      // this lane's positions p .. p+3
      const bool pok = p < m;                             // (m is a multiple of 4)
      double keep[FWD || G == 1 ? 1 : G - 1][2][4];       // BWD: sums of the groups so far
#pragma unroll
      for (int q = 0; q < G; ++q) {
        v4i acc[2][S];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int d = 0; d < S; ++d) acc[r][d] = (v4i){0, 0, 0, 0};
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          const int f = q * NKB + kb;
          const u4* src = bstep(jf, f + RD, jnext);
          u4 (&bc)[S] = b[f % RD];
          const u4* al = dig + (q * NKB + kb) * S * (DP / 16) + (pr * 32 + l16) * 4 + g;
          u4 xa[2][2];
#pragma unroll
          for (int r = 0; r < 2; ++r) xa[0][r] = al[r * 64];
#pragma unroll
          for (int i = 0; i < S; ++i) {
            if (i + 1 < S) {
#pragma unroll
              for (int r = 0; r < 2; ++r) xa[(i + 1) & 1][r] = al[(i + 1) * (DP / 16) + r * 64];
            }
#pragma unroll
            for (int s = S - 1 - i; s >= 0; --s)
#pragma unroll
              for (int r = 0; r < 2; ++r)
                acc[r][i + s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                    __builtin_bit_cast(v4i, bc[s]), __builtin_bit_cast(v4i, xa[i & 1][r]),
                    acc[r][i + s], 0, 0, 0);
            bc[S - 1 - i] = src[(S - 1 - i) * 64 + lane];
            // each digit's step stays in order: hoisted together, the loads
            // of many steps would not fit the registers
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        const int n = pok ? q * m + p : 0;                // FWD: the first mode
        const v4i f = *reinterpret_cast<const v4i*>(&sfx[n]);
        double vs[2][4];                                  // rows l16 and 16 + l16, positions p + v
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const int ex = sex[q][pr * 32 + r * 16 + l16];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            int d[S];
#pragma unroll
            for (int k = 0; k < S; ++k) d[k] = acc[r][k][v];
            vs[r][v] = oz_value<S>(d, ex, f[v]);
            // recombined here: left to the guarded stores below, every
            // group's integer sums would stay in registers until then
            if (!FWD && q + 1 < G) asm volatile("" : "+v"(vs[r][v]));
          }
        }
        if constexpr (FWD) {
          // this group's modes are final
          if (ghat) {
            const d4 lcn = *reinterpret_cast<const d4*>(&slc[n]);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              const bool ok = pok && rp + 16 * r < rows;
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const double rhat = vs[r][v];
                const double lam = srs[pr * 32 + 16 * r + l16] + lcn[v];
                const double val = rhat * ghat_fast(lam);
                fs0 += ok ? rhat * val : 0.0;
                fs1 += ok ? val * val : 0.0;
                fs2 += ok ? lam * (val * val) : 0.0;
                vs[r][v] = val;
              }
            }
          }
          if (a.gt) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              const double* gsrc =
                  a.gt + (uint32_t)(n * rows + (rp + 16 * r < rows ? rp + 16 * r + l16 : 0));
#pragma unroll
              for (int v = 0; v < 4; ++v) vs[r][v] *= gsrc[(uint32_t)(v * rows)];
            }
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) store(vs[0][v], vs[1][v], n + v, pok);
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            double y[G][2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              const double w = vs[r][v];
              if constexpr (G == 1) {
                y[0][r] = w;
              } else if constexpr (G == 2) {
                if (q == 0) {
                  keep[0][r][v] = w;
                } else {
                  y[0][r] = keep[0][r][v] + w;
                  y[1][r] = keep[0][r][v] - w;
                }
              } else {
                if (q == 0) {
                  keep[0][r][v] = w;
                } else if (q == 1) {
                  const double e = keep[0][r][v];
                  keep[0][r][v] = e + w;
                  keep[1][r][v] = e - w;
                } else if (q == 2) {
                  keep[2][r][v] = w;
                } else {
                  const double t0 = keep[2][r][v] + w, t1 = keep[2][r][v] - w;
                  y[0][r] = keep[0][r][v] + t0;
                  y[1][r] = keep[0][r][v] - t0;
                  y[2][r] = keep[1][r][v] + t1;
                  y[3][r] = keep[1][r][v] - t1;
                }
              }
            }
            if (q == G - 1) {
              const int h = K >> 1, pv = p + v;
              const int at[4] = {pv, K - 1 - pv, h - 1 - pv, h + pv};
#pragma unroll
              for (int o = 0; o < G; ++o) store(y[o][0], y[o][1], at[o], pok);
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    oz_load<G, FWD, PP, TPR>(row_src(tnext), K, m, tt, raw);
    if (FWD && a.rpart && (ghat || insum)) {
      // the tile's sums in a fixed order: lanes, then waves
      fs0 = wave_sum(fs0);
      fs1 = wave_sum(fs1);
      if (ghat) fs2 = wave_sum(fs2);
      if (lane == 0) {
        red[wave][0] = fs0;
        red[wave][1] = fs1;
        red[wave][2] = fs2;
      }
    }
    lds_barrier();                                        // the digits are consumed
    if (FWD && a.rpart && (ghat || insum) && tid == 0) {
      double t0 = 0.0, t1 = 0.0, t2 = 0.0;
      for (int w = 0; w < NW; ++w) {
        t0 += red[w][0];
        t1 += red[w][1];
        t2 += red[w][2];
      }
      if (ghat) {
        slot_ptr(a.rpart, rhs, S_DOT)[tile] = t0;
        slot_ptr(a.rpart, rhs, S_SUM)[tile] = 0.0;
        slot_ptr(a.rpart, rhs, S_SQ)[tile] = t1;
        slot_ptr(a.rpart, rhs, S_AUX2)[tile] = t2;
      } else {
        slot_ptr(a.rpart, rhs, S_TSUM)[tile] = t0;
        slot_ptr(a.rpart, rhs, S_TSQ)[tile] = t1;
      }
    }
  }
}

// Blocks per right-hand side: as many as fill the chip once (one or two per
// CU), never more than the tiles.
int oz_blocks(const OzGeom& q, int G, int S, int ntiles, int batch) {
  const size_t lds = (size_t)G * q.nkb * S * q.br * 64 + 8 * 1024;
  const int per_cu = q.nt == 512 ? 1 : (lds * 2 <= 160 * 1024 ? 2 : 1);
  return std::max(1, std::min(ntiles, (256 * per_cu + batch - 1) / batch));
}

template <int S, int G, bool FWD, int PP, int NT, int BR>
void oz_go(const OzGeom& q, const OzArgs& a, int batch, hipStream_t s) {
  const int nblk = oz_blocks(q, G, S, a.ntiles, batch);
  hipLaunchKernelGGL((mp_oz<S, G, FWD, PP, NT, BR>), dim3(nblk, batch), dim3(NT), 0, s, a);
}

template <int S, int G, bool FWD, int BR>
void oz_pairs(const OzGeom& q, const OzArgs& a, int batch, hipStream_t s) {
  const int ppg = q.pp * G;
  if constexpr (BR == 128) {                    // at most 32 points
    if (ppg == 4) oz_go<S, G, FWD, 4 / G, 256, BR>(q, a, batch, s);
    else oz_go<S, G, FWD, 8 / G, 256, BR>(q, a, batch, s);
  } else {
    switch (ppg) {
      case 4: oz_go<S, G, FWD, 4 / G, 256, BR>(q, a, batch, s); break;
      case 8: oz_go<S, G, FWD, 8 / G, 256, BR>(q, a, batch, s); break;
      case 12: oz_go<S, G, FWD, 12 / G, 256, BR>(q, a, batch, s); break;
      default: oz_go<S, G, FWD, 16 / G, 256, BR>(q, a, batch, s); break;
    }
  }
}

template <int S, int G, bool FWD>
void oz_pick(const OzGeom& q, const OzArgs& a, int batch, hipStream_t s) {
  if (q.nt == 512) {
    if (q.pp * G == 16) oz_go<S, G, FWD, 16 / G, 512, 32>(q, a, batch, s);
    else oz_go<S, G, FWD, 12 / G, 512, 32>(q, a, batch, s);
    return;
  }
  // (folding an axis this short would only pad: oz_fold_groups)
  if constexpr (G == 1) {
    if (q.br == 128) return oz_pairs<S, G, FWD, 128>(q, a, batch, s);
  }
  oz_pairs<S, G, FWD, 32>(q, a, batch, s);
}

template <int S>
void oz_groups(int G, bool fwd, const OzGeom& q, const OzArgs& a, int batch, hipStream_t s) {
  if (G == 4) return fwd ? oz_pick<S, 4, true>(q, a, batch, s) : oz_pick<S, 4, false>(q, a, batch, s);
  if (G == 2) return fwd ? oz_pick<S, 2, true>(q, a, batch, s) : oz_pick<S, 2, false>(q, a, batch, s);
  return fwd ? oz_pick<S, 1, true>(q, a, batch, s) : oz_pick<S, 1, false>(q, a, batch, s);
}

size_t oz_digit_bytes(int K, int G, int br, int S) {
  const OzGeom q = oz_geom(K, G, br);
  return (size_t)G * q.nf * q.nkb * S * 64 * 16;
}

}  // namespace

// Rows per tile for `rows` rows in all (the plan's largest batch).  A 16- or
// 32-point row is two threads' work in a tile of 128 rows and leaves most of a
// 32-row tile's threads and waves idle (K = 16, 282 k rows: 49 us in 32-row
// tiles, 25 in 128-row ones; K = 32, 64 of 32^3: 14 and 11).  From 48 points
// on 32-row tiles are the faster ones (48: 18 us against 23; 64: 30 against
// 34; 128: 36 against 40), as for few rows, which would leave CUs without a
// tile.
int oz_tile_rows(int K, int64_t rows) { return K <= 32 && rows / 128 >= 192 ? 128 : 32; }

// Parity groups of an int8 split product: the fewest matrix operations,
// padding included (64 slots a k-block, 16 columns a fragment), the fewer
// groups on a tie.
int oz_fold_groups(int K, int bc, int br) {
  auto cost = [&](int G) {
    const OzGeom q = oz_geom(K, G, br);
    return (int64_t)G * q.nkb * 64 * q.nf * 16;
  };
  int best = 1;
  if (bc != BC_DN && bc != BC_ND) {
    if (br == 32 && cost(2) < cost(best)) best = 2;
    if (br == 32 && bc == BC_P && cost(4) < cost(best)) best = 4;
  }
  return best;
}

int oz_partials(int64_t rows, int br) {
  const int64_t t = (rows + br - 1) / br;
  return t > (1 << 30) ? (1 << 30) : (int)t;
}

void launch_oz(const PinvOps& op, int ax, bool fwd, const void* X, void* Y, int batch,
               const RhsState* st, const double* la, const double* lb, const double* lc, int a1,
               const double* gt, double* rpart, hipStream_t s) {
  const int K = op.n[ax], G = op.fold[ax], br = op.br[ax], S = prec_digits(op.prec);
  const OzGeom q = oz_geom(K, G, br);
  const char* Bp = (const char*)(fwd ? op.Bf[ax] : op.Bb[ax]);
  OzArgs a{};
  a.B = (const u4*)Bp;
  a.fexp = (const int*)(Bp + oz_digit_bytes(K, G, br, S));
  a.X = (const double*)X;
  a.Y = (double*)Y;
  a.N = op.N;
  a.K = K;
  a.rows = (int)(op.N / K);
  a.m = K / G;
  a.nkb = q.nkb;
  a.nf = q.nf;
  a.ntiles = (a.rows + br - 1) / br;
  a.st = st;
  a.la = la;
  a.lb = lb;
  a.lc = lc;
  a.a1 = a1;
  a.gt = gt;
  a.rpart = rpart;
  if (S == 6) oz_groups<6>(G, fwd, q, a, batch, s);
  else oz_groups<7>(G, fwd, q, a, batch, s);
}

// Product q's kernel, as its template's name and total threads.
void oz_kernel_name(const PinvOps& op, int q, int batch, char* name, size_t len) {
  const int dim = op.dim, ax = q % dim, K = op.n[ax], G = op.fold[ax], br = op.br[ax];
  const int S = prec_digits(op.prec);
  const OzGeom g = oz_geom(K, G, br);
  const int blocks = oz_blocks(g, G, S, (int)((op.N / K + br - 1) / br), batch);
  snprintf(name, len, "kp::mp_oz<%d, %d, %s, %d, %d, %d>|%lld", S, G, q < dim ? "true" : "false",
           g.pp, g.nt, br, (long long)blocks * batch * g.nt);
}

size_t oz_packed_bytes(int K, int G, int br, int prec) {
  return oz_digit_bytes(K, G, br, prec_digits(prec)) + (size_t)K * sizeof(int);
}

// Packs the folded basis Qh (fold_basis: m x K, group-ordered columns) as the
// S digits read by mp_oz: for group q, column fragment jf, k-block kb, digit s
// and lane 16 g + c, 16 bytes hold digit s of column 16 jf + c at the k slots
// 64 kb + 16 g + 0..15, at (((q nf + jf) nkb + kb) S + s) 64 + lane.  Slot
// t (2 PP) + 2 c + e is position (forward) or mode (backward) 2 (c TPR + t) + e
// of the group.  Then the exponents f of the m columns of every group.  S = 7:
// the truncated base-128 digits of B 2^-f (max_k |B[k][n]| < 2^f).  S = 6: the
// balanced base-256 digits of the integer image trunc(B 2^(47 - f))
// (max_k |B[k][n]| < 2^f * 126/128), low to high; the digits in [-128, 127] of
// an integer are unique, so they are those the device takes from its data.
void oz_pack(const double* Qh, int K, int G, int br, bool fwd, int prec, void* dst) {
  const int S = prec_digits(prec), m = K / G;
  const OzGeom q = oz_geom(K, G, br);
  int8_t* o = (int8_t*)dst;                     // (zeroed by the caller)
  int* fx = (int*)(o + oz_digit_bytes(K, G, br, S));
  std::vector<int> slot(m);
  for (int k = 0; k < m; ++k) {
    const int pair = k / 2, c = pair / q.tpr, t = pair % q.tpr;
    slot[k] = t * 2 * q.pp + 2 * c + (k & 1);
  }
  for (int grp = 0; grp < G; ++grp)
    for (int n = 0; n < m; ++n) {
      auto at = [&](int k) {
        return fwd ? Qh[(size_t)k * K + grp * m + n] : Qh[(size_t)n * K + grp * m + k];
      };
      double mx = 0.0;
      for (int k = 0; k < m; ++k) mx = std::max(mx, std::fabs(at(k)));
      int f = 0;
      if (mx > 0.0) {
        const double fr = std::frexp(mx, &f);
        if (S == 6 && fr >= 0.984375) ++f;
      }
      fx[grp * m + n] = f;
      const double up = std::ldexp(1.0, S == 7 ? -f : 47 - f);
      for (int k = 0; k < m; ++k) {
        int dg[OZ_SMAX] = {0, 0, 0, 0, 0, 0, 0};
        double t = at(k) * up;                  // exact
        if (S == 7) {
          for (int d = 0; d < 7; ++d) {
            t *= 128.0;
            const double w = std::trunc(t);
            t -= w;
            dg[d] = (int)w;
          }
        } else {
          int64_t F = (int64_t)t;
          for (int d = 5; d >= 1; --d) {
            const int64_t w = ((F + 128) & 255) - 128;
            dg[d] = (int)w;
            F = (F - w) / 256;                  // exact
          }
          dg[0] = (int)F;                       // |F| <= 126
        }
        const int sl = slot[k], kb = sl / 64, lane = (sl % 64) / 16 * 16 + n % 16;
        for (int d = 0; d < S; ++d) {
          const size_t unit =
              ((((size_t)grp * q.nf + n / 16) * q.nkb + kb) * S + d) * 64 + lane;
          o[unit * 16 + sl % 16] = (int8_t)dg[d];
        }
      }
    }
}

}  // namespace kp
