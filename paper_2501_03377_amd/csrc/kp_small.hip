// Whole solves of small 2D problems in one kernel: Algorithm 1 with the FP64
// pseudoinverse preconditioner (Alg. 6), one 512-thread workgroup per
// right-hand side, every vector resident in LDS.
//
// For n x q grids up to 64 x 64 a solve is a few dozen tiny steps, so the
// multi-kernel path spends its time launching kernels.  Here P and two
// transform buffers (3 x 33 KiB) stay in LDS, R and U stay in registers, and
// the scalar recurrences, the stopping tests and the exit step (true residual,
// centring) run in the same kernel.
//
// One workgroup's chain of steps is bound by latency and by the FP64 matrix
// rate of a single CU (4096 cycles per plain 64 x 64 x 64 product), so
//   - a thread owns the points (x, y), (nx-1-x, y), (x, ny-1-y),
//     (nx-1-x, ny-1-y): it folds R by parity along both axes (kp_basis.cpp,
//     fold_basis, two groups) and unfolds Z in its registers, and each of the
//     four mode products is two half-size ones: half the matrix work;
//   - the products are in kp_fold.hip's packing, padded with zeros to whole
//     fragments, so no index is clamped and no value masked; a wave's operator
//     fragments are one or two 16-byte loads per four MFMAs, requested a
//     product ahead;
//   - every product reads X[r][k] along k and writes Y[n][r], so all four are
//     the same code.
// One iteration, against plain products of operators read element by element:
// 64 x 64 (D, D) 28.1 -> 17.8 us, (DN, ND) 45.4 -> 34.5, 33 x 50 24.1 -> 17.4,
// 5 x 7 14.4 -> 11.8; eight waves of eight points each do with a quarter fewer
// instructions than sixteen of four (22.2).
// The recurrences and stopping tests are those of the multi-kernel path,
// except that the low-mode certificate is not tried (the bound
// ||R|| / lambda_min or the estimate after the next application decide);
// the inner products, <R, Z> and the mean of Z included, are summed in space
// in a fixed order of their own, so results agree with that path to
// rounding.
#include <math.h>

#include "kp_common.h"
#include "kp_internal.h"

namespace kp {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int ST = 512;                  // threads per workgroup
constexpr int SW = ST / 64;              // waves
constexpr int SMAX = 64;                 // largest axis
constexpr int SE = 8;                    // points per thread
constexpr int TW = 2;                    // column tiles per wave in a product
// LDS row pitch in doubles: 16 rows 16 bytes each fall into distinct banks, and
// rows stay 16-byte aligned
constexpr int LP = SMAX + 2;
constexpr int SL = (SMAX + 1) * LP;      // doubles per grid buffer in LDS; the columns and
                                         // the row past SMAX hold the zero ghosts

// Lane moves of a double by DPP (two 32-bit halves) and reads of one lane.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double lane_d(double v, int l) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over the 16 lanes of each DPP row (pairs, quads, then two rotations);
// the first lane of a row holds the total in a fixed association.
__device__ __forceinline__ double row_sum(double v) {
  v += dpp<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp<0x124>(v);   // row_ror:4
  v += dpp<0x128>(v);   // row_ror:8
  return v;
}

// Fixed-order reduction of NV <= 4 values over the workgroup: the rows of each
// wave, then, for value q in lanes 16 q ..., the four row totals of a wave in
// order (lane % 16 takes a wave each) and one more row sum.  Every thread
// returns the same totals.  All lanes must be active.  `red` alternates
// between two buffers (turn), so that one barrier per sum is enough: a buffer
// is written again only after the next sum's barrier.
struct Red {
  double w[2][4][16][4];                 // [turn][value][wave][row]; waves past SW stay 0
};
template <int NV>
__device__ __forceinline__ void wg_sum(double (&v)[NV], Red& red, int& turn) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double (*r)[16][4] = red.w[turn];
  turn ^= 1;
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = row_sum(v[q]);
  if ((lane & 15) == 0)
#pragma unroll
    for (int q = 0; q < NV; ++q) r[q][wave][lane >> 4] = v[q];
  __syncthreads();
  const int q = lane >> 4;
  const double* p = r[q < NV ? q : 0][lane & 15];
  const d2 a = *reinterpret_cast<const d2*>(p), b = *reinterpret_cast<const d2*>(p + 2);
  const double t = row_sum((a.x + a.y) + (b.x + b.y));
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = lane_d(t, 16 * k);
}

__device__ __forceinline__ double ghat_s(double s) { return fabs(s) < 1e-13 ? 0.0 : 1.0 / s; }

// One axis of a product's operator: G groups of nb k-blocks and column
// fragments each (16 wide, padded).
struct Ax {
  int G, nb;
  __device__ __forceinline__ int tiles() const { return G * nb; }
};

// The operator fragments of a wave's column tiles.
template <int NB>
__device__ __forceinline__ void load_op(const u4* B, Ax a, u4 (&o)[TW][NB][2]) {
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const uint32_t ct = (wave >> 2) * TW + i;
    if (ct >= (uint32_t)a.tiles()) continue;
#pragma unroll
    for (int kb = 0; kb < NB; ++kb)
      if (kb < a.nb) {
        const u4* b = B + (ct * a.nb + kb) * 128;
        o[i][kb][0] = b[lane];
        o[i][kb][1] = b[lane + 64];
      }
  }
}

// Y[n][r] = sum_k X[r][k] B(k, n) (pitch LP) along axis a, whose group q
// contracts X's columns 16 nb q ...; the rows are `other`'s padded positions.
// Wave w owns rows 16 (w % 4) ... and the TW column tiles from TW (w / 4) on.
// The operator is the first MFMA operand: lane l supplies B(k, l % 16) and
// X(l % 16, k) with k = 4 (l / 16) + step of a k-block and receives
// Y(4 v + l / 16, l % 16).
template <int NB>
__device__ __forceinline__ void wg_gemm(const u4 (&o)[TW][NB][2], const double* X, double* Y,
                                        Ax a, Ax other, const double (*gh)[4]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rt = wave & 3, l16 = lane & 15, grp = lane >> 4;
  if (rt < other.tiles()) {
    const double* x = X + (rt * 16 + l16) * LP + 4 * grp;
    double* y = Y + grp * LP + rt * 16 + l16;
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const int ct = (wave >> 2) * TW + i;
      if (ct >= a.tiles()) continue;
      const double* xq = x + (a.G == 2 && ct >= a.nb ? 16 * a.nb : 0);
      d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kb = 0; kb < NB; ++kb)
        if (kb < a.nb) {
          const d2 x0 = *reinterpret_cast<const d2*>(xq + 16 * kb);
          const d2 x1 = *reinterpret_cast<const d2*>(xq + 16 * kb + 2);
          d2 b0, b1;
          __builtin_memcpy(&b0, &o[i][kb][0], 16);
          __builtin_memcpy(&b1, &o[i][kb][1], 16);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b0.x, x0.x, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b0.y, x0.y, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b1.x, x1.x, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b1.y, x1.y, acc, 0, 0, 0);
        }
#pragma unroll
      for (int v = 0; v < 4; ++v)
        y[(16 * ct + 4 * v) * LP] = gh ? acc[v] * gh[i][v] : acc[v];
    }
  }
  __syncthreads();
}

// Offsets along the axis (in positions) of the two neighbours of pos: the
// point itself at a wall whose ghost is the boundary cell, position SMAX, a
// zero, where the ghost is 0 (ghost rule of eq. 3.1).
__device__ __forceinline__ int lower(int pos, int n, int bc) {
  return pos > 0 ? -1 : (bc == BC_P ? n - 1 : ((bc == BC_D || bc == BC_DN) ? SMAX - pos : 0));
}
__device__ __forceinline__ int upper(int pos, int n, int bc) {
  return pos < n - 1 ? 1 : (bc == BC_P ? 1 - n : ((bc == BC_D || bc == BC_ND) ? SMAX - pos : 0));
}

// A value that every lane holds, kept in scalar registers.
__device__ __forceinline__ double uniform(double v) { return lane_d(v, 0); }

// NB: k-blocks per group of the longer axis, at most.
template <int NB>
__global__ __launch_bounds__(ST) void k_small_solve(Geom g, SmallOps o, const double* eta,
                                                    double* Uout, RhsState* st, RhsState* mirror,
                                                    double* hist, int hist_stride, double tol,
                                                    int max_iter, int flags) {
  __shared__ __attribute__((aligned(16))) double P[SL], TA[SL], TB[SL];
  __shared__ Red red;
  __shared__ RhsState rec;
  int turn = 0;
  const int rhs = blockIdx.x;
  const int nx = g.nx, ny = g.ny;
  const Ax ax = {o.G[0], o.nb[0]}, ay = {o.G[1], o.nb[1]};
  // this thread's points q: x mirrored for odd q, y for q & 2, the second
  // quadruple 16 rows on (a centre that is its own mirror image counts once)
  const int jx = threadIdx.x & 31, mx = nx - 1 - jx;
  const int jy[2] = {(int)(threadIdx.x >> 5), (int)(threadIdx.x >> 5) + 16};
  const int my[2] = {ny - 1 - jy[0], ny - 1 - jy[1]};
  const bool two_x = mx > jx, okx = mx >= jx;
  const double Nd = (double)g.N;
  const double* ep = eta + (int64_t)rhs * g.N;
  auto in = [&](int q) {
    return ((q & 1) ? two_x : okx) && ((q & 2) ? my[q >> 2] > jy[q >> 2] : my[q >> 2] >= jy[q >> 2]);
  };
  auto xq = [&](int q) { return (q & 1) ? mx : jx; };
  auto yq = [&](int q) { return (q & 2) ? my[q >> 2] : jy[q >> 2]; };
  auto li = [&](int q) { return yq(q) * LP + xq(q); };
  auto gi = [&](int q) { return in(q) ? (uint32_t)(yq(q) * nx + xq(q)) : 0u; };
  // its columns and rows in the transform buffers: the symmetric and the
  // antisymmetric group's, or the points' own
  auto slot = [&](int q) {
    return ((q & 1) && ax.G == 1 ? two_x : okx) &&
           ((q & 2) && ay.G == 1 ? my[q >> 2] > jy[q >> 2] : my[q >> 2] >= jy[q >> 2]);
  };
  auto ti = [&](int q) {
    const int c = (q & 1) ? (ax.G == 2 ? 16 * ax.nb + jx : mx) : jx;
    const int y = jy[q >> 2];
    return ((q & 2) ? (ay.G == 2 ? 16 * ay.nb + y : my[q >> 2]) : y) * LP + c;
  };
  // sums and differences along the folded axes, in place (both ways; a centre's
  // mirror image is 0 going in, its antisymmetric part comes out 0)
  auto fold = [&](double (&t)[SE]) {
#pragma unroll
    for (int h = 0; h < SE; h += 4) {
      if (ax.G == 2) {
        const double a = t[h], b = t[h + 1], c = t[h + 2], d = t[h + 3];
        t[h] = a + b; t[h + 1] = a - b; t[h + 2] = c + d; t[h + 3] = c - d;
      }
      if (ay.G == 2) {
        const double a = t[h], b = t[h + 1], c = t[h + 2], d = t[h + 3];
        t[h] = a + c; t[h + 2] = a - c; t[h + 1] = b + d; t[h + 3] = b - d;
      }
    }
  };
  double u[SE], r[SE];
#pragma unroll
  for (int q = 0; q < SE; ++q) u[q] = r[q] = 0.0;

  // the operator of the next product is requested before the running one; a
  // long unfolded axis leaves registers for one at a time
  constexpr int NO = NB == 2 ? 2 : 1;
  u4 op[NO][TW][NB][2];
  double e[SE];
#pragma unroll
  for (int q = 0; q < SE; ++q) e[q] = ep[gi(q)];
  if (NO == 2) load_op<NB>((const u4*)o.F[0], ax, op[0]);
  // Ghat of this lane's results of the second product (mode 16 ct + 4 v + grp
  // of y and 16 rt + l16 of x; past a group's last mode the product is 0)
  double gh[TW][4];
  {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double lx = o.l[0][(wave & 3) * 16 + (lane & 15)];
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        gh[i][v] = ghat_s(lx + o.l[1][((wave >> 2) * TW + i) * 16 + 4 * v + (lane >> 4)]);
  }
  // zeros where the transforms have no point or mode (products keep them), and
  // the zero ghosts
  for (int i = threadIdx.x; i < SL / 2; i += ST) {
    reinterpret_cast<d2*>(TA)[i] = (d2){0.0, 0.0};
    reinterpret_cast<d2*>(TB)[i] = (d2){0.0, 0.0};
    reinterpret_cast<d2*>(P)[i] = (d2){0.0, 0.0};
  }
  for (int i = threadIdx.x; i < (int)(sizeof(Red) / 8); i += ST) (&red.w[0][0][0][0])[i] = 0.0;
  __syncthreads();
  const int ox[2][2] = {{lower(jx, nx, g.bc[0]), upper(jx, nx, g.bc[0])},
                        {lower(mx, nx, g.bc[0]), upper(mx, nx, g.bc[0])}};
  int oy[4][2];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int y = (h & 1) ? my[h >> 1] : jy[h >> 1];
    oy[h][0] = lower(y, ny, g.bc[1]) * LP;
    oy[h][1] = upper(y, ny, g.bc[1]) * LP;
  }
  // minus Laplacian of the LDS grid p at point q (of this thread's)
  auto lap = [&](const double* p, int q) {
    const double* c = p + li(q);
    const int* a = ox[q & 1];
    const int* b = oy[q >> 1];
    return ((2.0 * c[0] - c[a[0]]) - c[a[1]]) + ((2.0 * c[0] - c[b[0]]) - c[b[1]]);
  };

  // the recurrences' scalars; those that are only reported go to `rec` (by
  // thread 0)
  struct {
    double h2, mean, rho, rsum, uu, rel_res;
    int iter, done, pinv_count;
  } s = {};
  const bool lead = threadIdx.x == 0;
  if (lead) rec = RhsState{};

  // R_0 = eta_c (eq. 3.6), since U_0 = 0
  {
    if (g.singular) {
      double v[1] = {0.0};
#pragma unroll
      for (int q = 0; q < SE; ++q)
        if (in(q)) v[0] += e[q];
      wg_sum<1>(v, red, turn);
      s.mean = uniform(v[0] / Nd);
    }
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < SE; ++q)
      if (in(q)) {
        r[q] = e[q] - s.mean;
        v[0] += r[q];
        v[1] += r[q] * r[q];
      }
    wg_sum<2>(v, red, turn);
    s.rsum = v[0];
    s.h2 = v[1];
    if (lead) rec.rr = v[1];
  }
  if (!isfinite(s.h2)) s.done = NONFINITE;
  else if (s.h2 == 0.0) s.done = ZERO_RHS;
  s.rel_res = s.done == ZERO_RHS ? 0.0 : 1.0;
  if (hist && threadIdx.x == 0) hist[(int64_t)rhs * hist_stride] = s.rel_res;

  // Z = M(R), rho, P = Z + beta P (centred, Remark 4.1), with the stopping
  // tests that follow an application
  auto precondition = [&](bool first) {
    // Z = M(R) (Alg. 6) from the folded R in TB back to TB; the operator of
    // each product is requested before the one ahead of it runs
    double z[SE];
#pragma unroll
    for (int q = 0; q < SE; ++q) z[q] = r[q];
    fold(z);
#pragma unroll
    for (int q = 0; q < SE; ++q)
      if (slot(q)) TB[ti(q)] = z[q];
    if (NO == 1 || !first) load_op<NB>((const u4*)o.F[0], ax, op[0]);
    if (NO == 2) load_op<NB>((const u4*)o.F[1], ay, op[NO - 1]);
    __syncthreads();
    wg_gemm<NB>(op[0], TB, TA, ax, ay, nullptr);        // F1[i][y']
    load_op<NB>((const u4*)(NO == 2 ? o.B[0] : o.F[1]), NO == 2 ? ax : ay, op[0]);
    wg_gemm<NB>(op[NO - 1], TA, TB, ay, ax, gh);        // F2[j][i]
    load_op<NB>((const u4*)(NO == 2 ? o.B[1] : o.B[0]), NO == 2 ? ay : ax, op[NO - 1]);
    wg_gemm<NB>(op[0], TB, TA, ax, ay, nullptr);        // G1[x'][j]
    if (NO == 1) load_op<NB>((const u4*)o.B[1], ay, op[0]);
    wg_gemm<NB>(op[NO - 1], TA, TB, ay, ax, nullptr);   // Z[y'][x']
#pragma unroll
    for (int q = 0; q < SE; ++q) z[q] = slot(q) ? TB[ti(q)] : 0.0;
    fold(z);
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < SE; ++q)
      if (in(q)) {
        v[0] += r[q] * z[q];
        v[1] += z[q];
        v[2] += z[q] * z[q];
      }
    wg_sum<3>(v, red, turn);
    const double zmean = g.singular ? v[1] / Nd : 0.0;
    const double rz = v[0] - zmean * s.rsum;
    double zz = v[2] - Nd * zmean * zmean;
    if (zz < 0.0) zz = 0.0;
    if (lead) {
      rec.zmean = zmean;
      rec.rz = rz;
      rec.zz = zz;
    }
    s.pinv_count += 1;
    if (!isfinite(rz) || !isfinite(zz)) { s.done = NONFINITE; return; }
    double beta = 0.0;
    if (first) {
      if (!(rz > 0.0)) { s.done = BREAKDOWN; return; }
      s.rho = uniform(rz);
    } else {
      const double err = s.uu > 0.0 ? sqrt(zz / s.uu) : INFINITY;
      if (lead) rec.err_est = err;
      if (!(flags & F_RESIDUAL_ONLY) && s.rel_res <= tol && err <= tol) {
        s.done = CONVERGED;
        return;
      }
      if (!(rz > 0.0)) { s.done = (s.rel_res <= tol) ? CONVERGED : BREAKDOWN; return; }
      beta = uniform(rz / s.rho);                            // beta_s = rho_s / rho_{s-1}
      s.rho = uniform(rz);
      if (lead) rec.beta = beta;
    }
#pragma unroll
    for (int q = 0; q < SE; ++q)
      if (in(q)) P[li(q)] = (z[q] - zmean) + (first ? 0.0 : beta * P[li(q)]);
    __syncthreads();
  };
  if (s.done == RUNNING) precondition(true);

  while (s.done == RUNNING && s.iter < max_iter) {
    // W_s = -Delta(P_{s-1}), alpha_s = rho_{s-1} / <W_s, P_{s-1}>
    double w[SE], alpha;
    {
      double v[1] = {0.0};
#pragma unroll
      for (int q = 0; q < SE; ++q) {
        w[q] = 0.0;
        if (in(q)) {
          w[q] = lap(P, q);
          v[0] += w[q] * P[li(q)];
        }
      }
      wg_sum<1>(v, red, turn);
      if (lead) rec.pw = v[0];
      if (!isfinite(v[0])) { s.done = NONFINITE; break; }
      if (!(v[0] > 0.0)) { s.done = BREAKDOWN; break; }
      alpha = uniform(s.rho / v[0]);
      if (lead) rec.alpha = alpha;
    }
    // U_s = U_{s-1} + alpha P, R_s = R_{s-1} - alpha W
    {
      double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < SE; ++q)
        if (in(q)) {
          u[q] += alpha * P[li(q)];
          r[q] -= alpha * w[q];
          v[0] += r[q];
          v[1] += r[q] * r[q];
          v[2] += u[q] * u[q];
        }
      wg_sum<3>(v, red, turn);
      s.rsum = v[0];
      s.uu = v[2];
      s.iter += 1;
      s.rel_res = uniform(sqrt(v[1] / s.h2));
      if (lead) rec.rr = v[1];
      if (hist && threadIdx.x == 0) hist[(int64_t)rhs * hist_stride + s.iter] = s.rel_res;
      if (!isfinite(s.rel_res)) { s.done = NONFINITE; break; }
      if (s.rel_res <= tol) {
        if (flags & F_RESIDUAL_ONLY) { s.done = CONVERGED; break; }
        // ||U_s - u|| = ||L^+ R_s|| <= ||R_s|| / lambda_min
        const double bound = v[2] > 0.0 ? sqrt(v[1] / v[2]) / g.lam_min : INFINITY;
        if (bound <= tol) {
          if (lead) rec.err_est = bound;
          s.done = CONVERGED;
          break;
        }
      }
    }
    precondition(false);
  }

  // exit step: true residual ||eta_c - L U|| / ||eta_c||, centring of U
  double true_rel, umean;
  {
#pragma unroll
    for (int q = 0; q < SE; ++q) e[q] = ep[gi(q)];   // (again: not kept over the products)
#pragma unroll
    for (int q = 0; q < SE; ++q)
      if (in(q)) TA[li(q)] = u[q];
    __syncthreads();
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < SE; ++q)
      if (in(q)) {
        const double t = (e[q] - s.mean) - lap(TA, q);
        v[0] += t * t;
        v[1] += u[q];
      }
    wg_sum<2>(v, red, turn);
    true_rel = s.h2 > 0.0 ? sqrt(v[0] / s.h2) : 0.0;
    umean = g.singular ? v[1] / Nd : 0.0;
#pragma unroll
    for (int q = 0; q < SE; ++q)
      if (in(q)) Uout[(int64_t)rhs * g.N + gi(q)] = u[q] - umean;
  }
  if (lead) {
    RhsState out = rec;
    out.h2 = s.h2;
    out.mean = s.mean;
    out.rho = s.rho;
    out.rsum = s.rsum;
    out.uu = s.uu;
    out.rel_res = s.rel_res;
    out.true_rel_res = true_rel;
    out.umean = umean;
    out.scale = out.inv_scale = 1.0;
    out.iter = s.iter;
    out.done = s.done;
    out.pinv_count = s.pinv_count;
    out.diag_iter = -1;
    st[rhs] = out;
    if (mirror) mirror[rhs] = out;
  }
}

}  // namespace

bool small_solve_fits(const Geom& g) { return g.dim == 2 && g.nx <= SMAX && g.ny <= SMAX; }

void launch_small_solve(const Geom& g, const SmallOps& o, const double* eta, double* U,
                        RhsState* st, RhsState* mirror, double* hist, int hist_stride, int batch,
                        double tol, int max_iter, int flags, hipStream_t s) {
  trace_begin(KC_SMALL, s);
  // two k-blocks per group hold 32 points, every folded axis; an unfolded one
  // of more than that has up to four
  if (o.nb[0] <= 2 && o.nb[1] <= 2)
    hipLaunchKernelGGL(k_small_solve<2>, dim3(batch), dim3(ST), 0, s, g, o, eta, U, st, mirror,
                       hist, hist_stride, tol, max_iter, flags);
  else
    hipLaunchKernelGGL(k_small_solve<4>, dim3(batch), dim3(ST), 0, s, g, o, eta, U, st, mirror,
                       hist, hist_stride, tol, max_iter, flags);
  trace_end(KC_SMALL, s);
}

}  // namespace kp
