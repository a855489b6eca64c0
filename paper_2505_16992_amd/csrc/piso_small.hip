// Whole Krylov solves of small grids in one work-group.
//
// The solves of a 32 x 32 step were some 150 kernels of 3 - 6 us on one or a few CUs: nothing
// but launches, partial sums through memory and pipeline fills.  Up to kSmallCells cells the
// vectors of a solve fit one work-group's registers, and the operand of the stencil, the
// transformed fields and (where there is room) the bases its LDS.  What bounds an iteration is
// then the latency of its eight (PCG) or five (BiCGStab) phases between barriers: 2.5 us (18 x
// 16, FP32) to 5.3 us (49 x 17, FP64) for one of the PCG, 21 us by launches; 2.2 - 2.6 us for
// one of the BiCGStab, 19 us by launches.  The arithmetic is that of the kernels it stands
// for (piso_krylov.hip, piso_fdm.hip): the same recurrences, tests of convergence and
// breakdown, FP64 sums.  The vectors are FP64 in both types: it costs next to nothing here, and
// what FP32 solves leave is then the tolerance and the rounding of the stored fields.
//
// Each thread owns CPT cells.  The coefficients and neighbours of its cells are read once; a
// cell beyond the grid has coefficients 0 and vectors 0.  The state goes to the device copy
// and to the host's pinned one, so that a solve is one launch and one wait.
#include <cmath>
#include <string>

#include "piso_impl.h"
#include "piso_mma.h"

namespace piso {

namespace {

// BiCGStab: one wave per SIMD, since every wave repeats the scalar work between the sums (8
// waves took 3.0 - 3.2 us an iteration on 18 x 16 to 49 x 17 cells where 4 take 2.2 - 2.6).
// PCG: two, whose products hide each other's latencies.
constexpr int kBiWG = 256, kPcgWG = 512;

// Sums of NV <= 8 values over a work-group of at most WG threads, the same in every thread, in
// a fixed order: rows of 16 lanes, then the rows' sums of several values at a time.  One
// barrier a call: successive calls alternate between the two halves of red, zeroed where the
// work-group has fewer rows.
template <int WG>
struct SmallSum {
  static constexpr int ROWS = WG / 16, PER = 64 / ROWS;   // values a wave re-reduces at a time
  double* red;                                            // LDS [2][8][ROWS]
  int half;
  __device__ __forceinline__ void init(double* r) {
    red = r;
    half = 0;
    for (int e = threadIdx.x; e < 2 * 8 * ROWS; e += blockDim.x) r[e] = 0.0;
    __syncthreads();
  }
  template <int NV>
  __device__ __forceinline__ void operator()(double (&v)[NV]) {
    static_assert(NV <= 8 && (ROWS == 16 || ROWS == 32), "rows of 16 lanes");
    const int lane = threadIdx.x & 63, row = threadIdx.x >> 4;
    double* p = red + half * 8 * ROWS;
    half ^= 1;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const double t = row_sum(v[q]);
      if ((lane & 15) == 0) p[q * ROWS + row] = t;
    }
    __syncthreads();
#pragma unroll
    for (int q0 = 0; q0 < NV; q0 += PER) {
      const double t = row_sum(p[q0 * ROWS + lane]);
#pragma unroll
      for (int q = q0; q < NV && q < q0 + PER; ++q) {
        v[q] = lane_value(t, (q - q0) * ROWS);
        if constexpr (ROWS == 32) v[q] += lane_value(t, (q - q0) * ROWS + 16);
      }
    }
  }
};

}  // namespace

// ------------------------------------------------------------------------- BiCGStab

// Jacobi BiCGStab of D right-hand sides (C^T with TRANS).  Shared: the operand of C K^-1.
template <typename R, int D, bool TRANS, int CPT>
__global__ void __launch_bounds__(kBiWG)
k_bi_small(Grid g, const R* __restrict__ A, const R* __restrict__ C, const R* __restrict__ b, R* __restrict__ x,
           int from_zero, BiState* st, BiState* host, unsigned long long seq, double tol2, int max_iter) {
  extern __shared__ __align__(32) char smem[];
  __shared__ double red[2 * 8 * kBiWG / 16];
  double* op = (double*)smem;   // [D][N]
  SmallSum<kBiWG> sum;
  sum.init(red);
  const int N = g.N, nth = blockDim.x;
  double a[CPT][2 * D], iA[CPT], xv[CPT][D], r[CPT][D], rh[CPT][D], p[CPT][D], v[CPT][D];
  int F[CPT][2 * D], cell[CPT];
  double t0[2 * D], bb[D], rr[D], rho[D], rho_old[D], alpha[D], omega[D];
#pragma unroll
  for (int c = 0; c < 2 * D; ++c) t0[c] = 0.0;
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    const int P0 = (int)threadIdx.x + u * nth;
    const bool on = P0 < N;
    const int P = on ? P0 : 0;
    cell[u] = on ? P : -1;
    const Cell cl = locate(g, P);
#pragma unroll
    for (int f = 0; f < 2 * D; ++f) {
      const int j = f >> 1, Q = neighbour(g, cl, P, j, f & 1);
      const int Qc = Q >= 0 ? Q : P;
      // coefficient of the neighbour: (C or C^T)_{P Q}; slot j: upper, D + j: lower neighbour
      const R cv = (f & 1) ? (TRANS ? C[(size_t)(D + j) * N + P] : C[(size_t)j * N + P])
                           : (TRANS ? C[(size_t)j * N + Qc] : C[(size_t)(D + j) * N + Qc]);
      F[u][f] = Qc;
      a[u][f] = on && Q >= 0 ? (double)cv : 0.0;
    }
    const double AP = A[P];
    iA[u] = 1.0 / AP;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      const R* xc = x + (size_t)c * N;
      xv[u][c] = on && !from_zero ? (double)xc[P] : 0.0;
      double Cx = AP * xv[u][c];
      if (!from_zero) {
#pragma unroll
        for (int f = 0; f < 2 * D; ++f) Cx += a[u][f] * (double)xc[F[u][f]];
      }
      const double bv = on ? (double)b[(size_t)c * N + P] : 0.0;
      const double rv = on ? bv - Cx : 0.0;
      r[u][c] = rh[u][c] = rv;
      p[u][c] = v[u][c] = 0.0;
      t0[c] += rv * rv;
      t0[D + c] += bv * bv;
    }
    if (on) op[P] = iA[u];
  }
  sum(t0);
#pragma unroll
  for (int u = 0; u < CPT; ++u)   // the neighbours' K^-1
#pragma unroll
    for (int f = 0; f < 2 * D; ++f) a[u][f] *= op[F[u][f]];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < D; ++c) {
    rho[c] = rr[c] = t0[c];
    bb[c] = t0[D + c];
  }
  int done[D], iters[D], status[D];
  double rlast[D];
#pragma unroll
  for (int c = 0; c < D; ++c) {
    rho_old[c] = alpha[c] = omega[c] = 1.0;
    status[c] = iters[c] = done[c] = 0;
    rlast[c] = rr[c];
    if (!std::isfinite(rr[c]) || !std::isfinite(bb[c])) {
      status[c] = PISO_E_NAN;
      done[c] = 1;
    } else if (bb[c] == 0.0 || rr[c] <= tol2 * bb[c]) {
      done[c] = 1;
    }
    if (bb[c] == 0.0) {
#pragma unroll
      for (int u = 0; u < CPT; ++u) xv[u][c] = 0.0;
    }
  }
  // y = C K^-1 z for the components still active; z in LDS for the neighbours
  auto apply = [&](double(&z)[CPT][D], double(&y)[CPT][D]) {
#pragma unroll
    for (int u = 0; u < CPT; ++u)
      if (cell[u] >= 0) {
#pragma unroll
        for (int c = 0; c < D; ++c) op[c * N + cell[u]] = z[u][c];
      }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < CPT; ++u)
#pragma unroll
      for (int c = 0; c < D; ++c) {
        double t = z[u][c];
#pragma unroll
        for (int f = 0; f < 2 * D; ++f) t += a[u][f] * op[c * N + F[u][f]];
        y[u][c] = t;
      }
  };
  for (int k = 0;; ++k) {
    int live = 0;
    double beta[D], om[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      beta[c] = om[c] = 0.0;
      if (done[c]) continue;
      const bool conv = rr[c] <= tol2 * bb[c];
      const bool bad = !std::isfinite(rho[c]) || !std::isfinite(rr[c]);
      const bool brk = k < max_iter && !conv && !bad && omega[c] == 0.0;
      rlast[c] = rr[c];
      if (k > 0) iters[c] = k;
      if (conv || bad || brk) {
        status[c] = bad ? PISO_E_NAN : (brk ? PISO_BREAKDOWN : 0);
        done[c] = 1;
        continue;
      }
      beta[c] = rho[c] * alpha[c] / (rho_old[c] * omega[c]);
      om[c] = omega[c];
      if (rho[c] == 0.0) {   // r orthogonal to rh to the last bit: go on from r as a new start
        beta[c] = 0.0;
        rho[c] = rr[c];
#pragma unroll
        for (int u = 0; u < CPT; ++u) rh[u][c] = r[u][c];
      }
      rho_old[c] = rho[c];
      ++live;
    }
    if (live == 0 || k >= max_iter) break;
    double t[CPT][D];
#pragma unroll
    for (int u = 0; u < CPT; ++u)
#pragma unroll
      for (int c = 0; c < D; ++c)
        if (!done[c]) p[u][c] = r[u][c] + beta[c] * (p[u][c] - om[c] * v[u][c]);
    apply(p, v);
    double rv[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      rv[c] = 0.0;
#pragma unroll
      for (int u = 0; u < CPT; ++u) rv[c] += rh[u][c] * v[u][c];
    }
    sum(rv);
    live = 0;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      if (done[c]) continue;
      if (rv[c] == 0.0 || !std::isfinite(rv[c])) {
        status[c] = std::isfinite(rv[c]) ? PISO_BREAKDOWN : PISO_E_NAN;
        iters[c] = k;
        done[c] = 1;
        continue;
      }
      alpha[c] = rho[c] / rv[c];
      ++live;
    }
    if (live == 0) break;
#pragma unroll
    for (int u = 0; u < CPT; ++u)   // s takes r's place
#pragma unroll
      for (int c = 0; c < D; ++c)
        if (!done[c]) r[u][c] -= alpha[c] * v[u][c];
    apply(r, t);
    double ts[2 * D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      ts[c] = ts[D + c] = 0.0;
#pragma unroll
      for (int u = 0; u < CPT; ++u) {
        const double tv = cell[u] >= 0 ? t[u][c] : 0.0;
        ts[c] += tv * r[u][c];
        ts[D + c] += tv * tv;
      }
    }
    sum(ts);
    double nx[2 * D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      nx[c] = nx[D + c] = 0.0;
      if (done[c]) continue;
      omega[c] = ts[D + c] > 0.0 ? ts[c] / ts[D + c] : 0.0;
      const double al = alpha[c], w = omega[c];
#pragma unroll
      for (int u = 0; u < CPT; ++u) {
        xv[u][c] += (al * p[u][c] + w * r[u][c]) * iA[u];
        r[u][c] -= w * t[u][c];
        nx[c] += rh[u][c] * r[u][c];
        nx[D + c] += r[u][c] * r[u][c];
      }
    }
    sum(nx);
#pragma unroll
    for (int c = 0; c < D; ++c) {
      if (done[c]) continue;
      rho[c] = nx[c];
      rr[c] = nx[D + c];
    }
  }
#pragma unroll
  for (int u = 0; u < CPT; ++u)
    if (cell[u] >= 0) {
#pragma unroll
      for (int c = 0; c < D; ++c) x[(size_t)c * N + cell[u]] = (R)xv[u][c];
    }
  // every wave's part of x is in the L2 before the state is published, whose release writes
  // that back (a device fence by every wave took 1.2 us)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    BiState o{};
    o.tol2 = tol2;
    o.all_done = 1;
    for (int c = 0; c < 3; ++c) o.done[c] = 1;
#pragma unroll
    for (int c = 0; c < D; ++c) {
      o.rr[c] = rlast[c];
      o.bb[c] = bb[c];
      o.done[c] = done[c];
      o.iters[c] = iters[c];
      o.status[c] = status[c];
      o.all_done &= done[c];
    }
    *st = o;
    o.seq = seq - 1;
    *host = o;
    publish(&host->seq, seq);
  }
}

// ------------------------------------------------------ PCG with fast diagonalisation

// The 2D preconditioner's plan (piso_fdm_plan.h, piso_fdm.hip); positions are row-major in the
// box, n0 a row, n1 rows.
template <typename R>
struct SmallFdm {
  int n0, n1, t0, t1, ld, line;   // t: tiles of 16; ld: LDS row
  const int* map;
  int rowfast;
  const R *f0, *i0, *f1, *i1;     // packed bases of x and (without a line) y
  const R *l0, *l1;               // eigenvalues
  const double* ones;
  const FdmSel* sel;
  const double* k;                // couplings along the line
  const R* piv;                   // reciprocal pivots [n1][n0]
};

// One product on the matrix cores: COL false, Y[r][m] = sum_k V[k][m] X[r][k]; true,
// Y[m][c] = sum_k V[k][m] X[k][c].  X and Y are [16 t1][ld], zero beyond the box (the packed
// basis is zero there too, so that it stays so).  each(row, col, value) passes the results on.
template <typename R, bool COL, typename Fn>
__device__ __forceinline__ void small_product(const SmallFdm<R>& a, const R* V, const R* X, Fn&& each) {
  using V4 = typename Vec4<R>::T;
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int g = lane >> 4, nl = lane & 15;
  const int kc = COL ? a.t1 : a.t0, mt = kc, tt = COL ? a.t0 : a.t1;
  const bool one = (COL ? a.n1 : a.n0) == 16 * (kc - 1) + 1;   // one row in the last tile: in step 0
  int m = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = 0;   // output tile of this wave
  for (;; m += nw) {
    while (m >= mt) {
      m -= mt;
      ++t;
    }
    if (t >= tt) break;
    V4 acc = V4{R(0), R(0), R(0), R(0)};
    const R* vp = V + ((size_t)m * kc * 64 + lane) * 4;
    const R* xp = COL ? X + 4 * g * a.ld + t * 16 + nl : X + (t * 16 + nl) * a.ld + 4 * g;
    auto load = [&](int k, V4& av, V4& bv) {
      av = *reinterpret_cast<const V4*>(vp + k * 256);
      if constexpr (COL) {
#pragma unroll
        for (int u = 0; u < 4; ++u) bv[u] = xp[(k * 16 + u) * a.ld];
      } else {
        bv = lds4<R>(xp + k * 16);
      }
    };
    V4 av, bv;
    load(0, av, bv);
    for (int k = 1; k < kc; ++k) {
      V4 an, bn;
      load(k, an, bn);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = mma(av[u], bv[u], acc);
      av = an;
      bv = bn;
    }
    acc = mma(av[0], bv[0], acc);
    if (!one) {
#pragma unroll
      for (int u = 1; u < 4; ++u) acc = mma(av[u], bv[u], acc);
    }
    each(m * 16 + 4 * g, t * 16 + nl, acc);
  }
}

// STAGE: the bases in LDS.
template <typename R, int CPT, bool STAGE>
__global__ void __launch_bounds__(kPcgWG)
k_pcg_small(Grid g, SmallFdm<R> a, const R* __restrict__ Pf, const R* __restrict__ bsrc,
            const double* __restrict__ mean, double sign, const R* x0, R* x, int gauge, double tol2, double met2,
            int max_k, CgState* st, CgState* host, unsigned long long seq) {
  using V4 = typename Vec4<R>::T;
  extern __shared__ __align__(32) char smem[];
  __shared__ double red[2 * 8 * kPcgWG / 16];
  __shared__ double rmean;   // mean of the residual last transformed
  const int N = g.N, nth = blockDim.x, tile = 16 * a.t1 * a.ld;
  double* dS = (double*)smem;             // [N] direction, by cell
  R* X = (R*)(dS + (N + 3) / 4 * 4);      // [16 t1][ld]
  R* Y = X + tile;                        // [16 t1][ld]
  R* l1 = Y + tile;                       // [16 t1] the line's couplings
  R* I = l1 + 16 * a.t1;             // [16 t1][ld] reciprocal pivots, or eigenvalues of the inverse
  const int ldi = a.ld;
  SmallSum<kPcgWG> sum;
  const int q = a.sel->q, rejected = a.sel->bad;
  const int b0 = a.t0 * a.t0 * 256, b1 = a.line ? 0 : a.t1 * a.t1 * 256;
  const R* f0 = a.f0 + (size_t)q * b0;
  const R* i0 = a.i0 + (size_t)q * b0;
  const R* f1 = a.line ? nullptr : a.f1 + (size_t)q * b1;
  const R* i1 = a.line ? nullptr : a.i1 + (size_t)q * b1;
  if constexpr (STAGE) {
    R* B = I + tile;
    for (int e = 4 * (int)threadIdx.x; e < b0; e += 4 * nth) {
      *reinterpret_cast<V4*>(B + e) = *reinterpret_cast<const V4*>(f0 + e);
      *reinterpret_cast<V4*>(B + b0 + e) = *reinterpret_cast<const V4*>(i0 + e);
    }
    f0 = B;
    i0 = B + b0;
    B += 2 * b0;
    for (int e = 4 * (int)threadIdx.x; e < b1; e += 4 * nth) {
      *reinterpret_cast<V4*>(B + e) = *reinterpret_cast<const V4*>(f1 + e);
      *reinterpret_cast<V4*>(B + b1 + e) = *reinterpret_cast<const V4*>(i1 + e);
    }
    f1 = B;
    i1 = B + b1;
  }
  const double ones = a.ones[q];
  for (int e = threadIdx.x; e < 2 * tile; e += nth) X[e] = R(0);
  if (a.line) {
    for (int e = threadIdx.x; e < a.n1; e += nth) l1[e] = (R)a.k[e];
  } else {   // the null mode, and what is beyond the box, is left out
    for (int e = threadIdx.x; e < tile; e += nth) I[e] = R(0);
    __syncthreads();
  }
  sum.init(red);
  const double mu = mean ? mean[0] : 0.0;
  double c[CPT][4], xv[CPT], r[CPT], d[CPT], z[CPT];
  int F[CPT][4], cell[CPT], at[CPT];
  double t2[2] = {0.0, 0.0};
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    const int e0 = (int)threadIdx.x + u * nth;
    const bool on = e0 < N;
    const int e = on ? e0 : 0, row = e / a.n0, col = e - row * a.n0;
    const int P = a.map ? a.map[a.rowfast ? (size_t)col * a.n1 + row : (size_t)e] : e;
    cell[u] = on ? P : -1;
    at[u] = row * a.ld + col;
    if (on) {
      if (a.line) {
        I[at[u]] = a.piv[e];
      } else {
        const R l = a.l1[q * a.n1 + row] + a.l0[q * a.n0 + col];
        I[at[u]] = l > R(0) ? R(1) / l : R(0);
      }
    }
    const Cell cl = locate(g, P);
    xv[u] = on && x0 ? (double)x0[P] : 0.0;   // null: from zero
    double Mx = 0.0;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const int j = f >> 1, Q = neighbour(g, cl, P, j, f & 1), Qc = Q >= 0 ? Q : P;
      const double pf = Pf[(size_t)j * N + ((f & 1) ? P : Qc)];
      F[u][f] = Qc;
      c[u][f] = on && Q >= 0 ? pf : 0.0;
      if (x0) Mx += c[u][f] * (xv[u] - (double)x0[Qc]);
    }
    const double bv = on ? sign * ((double)bsrc[P] - mu) : 0.0;
    r[u] = bv - Mx;
    d[u] = z[u] = 0.0;
    t2[0] += r[u] * r[u];
    t2[1] += bv * bv;
  }
  sum(t2);
  double rr = t2[0], rr_old = rr, rz = 0.0, rz_old = 1.0;
  const double bb = t2[1];
  int k = 0, status = 0;
  bool done = false;
  const double tol2bb = tol2 * bb, met2bb = met2 * bb;
  if (!std::isfinite(rr) || !std::isfinite(bb)) {
    status = PISO_E_NAN;
    done = true;
  } else if (bb == 0.0 || rr <= tol2 * bb) {
    done = true;
  } else if (rejected) {   // the host runs the solve with multigrid
    status = kFdmRejected;
    done = true;
  }
  if (bb == 0.0) {
#pragma unroll
    for (int u = 0; u < CPT; ++u) xv[u] = 0.0;
  }
  // z = B r, the residual freed of its mean, and r.z, r.r.  B works in R, in FP32 on residuals of
  // norms below 1e-30 times a power of two (B is linear; the transforms of residuals below 1e-37
  // would lose their digits: 18 x 16 cells, right-hand sides of 2e-38, stayed at 2.7e-7).
  auto precondition = [&]() {
    const bool scaled = sizeof(R) == 4 && __builtin_amdgcn_readfirstlane(rr < 1e-60);
#pragma unroll
    for (int u = 0; u < CPT; ++u)
      if (cell[u] >= 0) X[at[u]] = scaled ? (R)(r[u] * 0x1p100) : (R)r[u];
    __syncthreads();
    auto store_row = [&](R* D) {
      return [&, D](int col, int row, V4 v) { sts4<R>(D + row * a.ld + col, v); };
    };
    small_product<R, false>(a, f0, X, store_row(Y));
    __syncthreads();
    if (a.line) {
      // column c of Y: a tridiagonal system along the rows, two lanes a column from both ends
      // to the middle row; the null mode (column 0) without its means
      const int n = a.n1, m = n / 2, lane = threadIdx.x & 63, half = lane >> 5;
      const int steps = half ? n - 1 - m : m;
      for (int c0 = (int)(threadIdx.x >> 6) * 32; c0 < a.n0; c0 += nth >> 1) {
        const bool on = c0 + (lane & 31) < a.n0;
        const int cc = on ? c0 + (lane & 31) : a.n0 - 1;
        const R* Ic = I + cc;
        R* Yc = Y + cc;
        R off = R(0);
        if (c0 == 0) {
          double t = 0.0;
          for (int j = lane; j < n; j += 64) t += (double)Y[j * a.ld];
          t = wave_sum(t);
          if (lane == 0) rmean = t * ones;
          off = (lane & 31) == 0 ? (R)(t / n) : R(0);
        }
        // four rows' reads at a time, ahead of the chain
        auto rows = [&](int s0, bool fwd, auto&& fn) {
          R y[4], iv[4], kk[4];
          int jj[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int t = fwd ? min(s0 + u, steps - 1) : max(s0 - u, 0);
            const int j = jj[u] = half ? n - 1 - t : t;
            y[u] = Yc[j * a.ld];
            iv[u] = Ic[j * a.ld];
            kk[u] = l1[half ? j - 1 : j];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (fwd ? s0 + u < steps : s0 - u >= 0) {
              const R w = fn(y[u], iv[u], kk[u]);
              if (on) Yc[jj[u] * a.ld] = w;
            }
        };
        R v = R(0), f = R(0);   // value and factor k / p of the row before
        for (int s = 0; s < steps; s += 4)
          rows(s, true, [&](R y, R iv, R kk) {
            v = (y - off) + f * v;
            f = kk * iv;
            return v;
          });
        const R mine = f * v;
        const R other = __shfl_xor(mine, 32, 64);
        R w = ((Yc[m * a.ld] - off) + (half ? other + mine : mine + other)) * Ic[m * a.ld];
        if (half == 0 && on) Yc[m * a.ld] = w;
        double tot = half == 0 ? (double)w : 0.0;
        for (int s = steps - 1; s >= 0; s -= 4)
          rows(s, false, [&](R y, R iv, R kk) {
            w = y * iv + (kk * iv) * w;
            tot += (double)w;
            return w;
          });
        if (c0 == 0) {   // the null mode's solution without its mean
          const R shift = (R)((lane_value(tot, 0) + lane_value(tot, 32)) / n);
          for (int j = lane; j < n; j += 64) Y[j * a.ld] -= shift;
        }
      }
      __syncthreads();
    } else {
      small_product<R, true>(a, f1, Y, [&](int row, int col, V4 v) {
        if (row == 0 && col == 0) rmean = (double)v[0] * ones;
#pragma unroll
        for (int u = 0; u < 4; ++u) X[(row + u) * a.ld + col] = v[u] * I[(row + u) * a.ld + col];
      });
      __syncthreads();
      small_product<R, true>(a, i1, X, [&](int row, int col, V4 v) {
#pragma unroll
        for (int u = 0; u < 4; ++u) Y[(row + u) * a.ld + col] = v[u];
      });
      __syncthreads();
    }
    small_product<R, false>(a, i0, Y, store_row(X));
    __syncthreads();
    const double off = scaled ? rmean * 0x1p-100 : rmean;
    double t[2] = {0.0, 0.0};
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      if (cell[u] < 0) continue;
      z[u] = (double)X[at[u]];
      if (scaled) z[u] *= 0x1p-100;
      r[u] -= off;
      t[0] += r[u] * z[u];
      t[1] += r[u] * r[u];
    }
    sum(t);
    rz = t[0];
    rr = t[1];
  };
  while (!done) {
    precondition();
    if (!std::isfinite(rz) || !std::isfinite(rr)) {
      status = PISO_E_NAN;
      break;
    }
    if (rr <= tol2bb || (k > 0 && rr <= met2bb && rr >= rr_old)) break;
    rr_old = rr;
    if (k >= max_k) {
      status = PISO_NOT_CONVERGED;
      break;
    }
    const double beta = k == 0 ? 0.0 : rz / rz_old;
    rz_old = rz;
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      d[u] = z[u] + beta * d[u];
      if (cell[u] >= 0) dS[cell[u]] = d[u];
    }
    __syncthreads();
    double t[1] = {0.0};
#pragma unroll
    for (int u = 0; u < CPT; ++u) {   // q takes z's place
      double Md = 0.0;
#pragma unroll
      for (int f = 0; f < 4; ++f) Md += c[u][f] * (d[u] - dS[F[u][f]]);
      z[u] = Md;
      t[0] += d[u] * Md;
    }
    sum(t);
    if (!(t[0] > 0.0) || !std::isfinite(t[0])) {
      status = std::isfinite(t[0]) ? PISO_BREAKDOWN : PISO_E_NAN;
      break;
    }
    const double alpha = rz / t[0];
    ++k;
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      xv[u] += alpha * d[u];
      r[u] -= alpha * z[u];
    }
  }
  if (status != kFdmRejected) {
    double off = 0.0;
    if (gauge) {
      double t[1] = {0.0};
#pragma unroll
      for (int u = 0; u < CPT; ++u) t[0] += xv[u];
      sum(t);
      off = t[0] / N;
    }
#pragma unroll
    for (int u = 0; u < CPT; ++u)
      if (cell[u] >= 0) x[cell[u]] = (R)(xv[u] - off);
  }
  if (threadIdx.x == 0) {
    CgState o{};
    o.rr = rr;
    o.bb = bb;
    o.tol2 = tol2;
    o.met2 = met2;
    o.done = 1;
    o.iters = o.k = k;
    o.max_k = max_k;
    o.status = status;
    o.zero_rhs = bb == 0.0 ? 1 : 0;
    *st = o;
    answer(host, o, seq);
  }
}

// ------------------------------------------------------------------------------ host

namespace {

int small_check(piso_ctx* c, hipStream_t s, const unsigned long long* seq, const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(c, PISO_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
  return wait_pinned(c, s, seq, what);
}

int small_threads(int N, int wg) { return std::min(wg, (N + 63) / 64 * 64); }

template <typename R>
SmallFdm<R> small_fdm(const piso_ctx* c) {
  const FdmState& f = c->fdm;
  SmallFdm<R> a{};
  a.n0 = f.n[0];
  a.n1 = f.n[1];
  a.t0 = (a.n0 + 15) / 16;
  a.t1 = (a.n1 + 15) / 16;
  a.ld = 16 * a.t0 + 4;
  a.line = f.line >= 0 ? 1 : 0;
  a.map = f.map;
  a.rowfast = f.rowfast;
  a.f0 = (const R*)f.fwd[0];
  a.i0 = (const R*)f.inv[0];
  a.f1 = (const R*)f.fwd[1];
  a.i1 = (const R*)f.inv[1];
  a.l0 = (const R*)f.lam[0];
  a.l1 = (const R*)f.lam[1];
  a.ones = f.ones;
  a.sel = f.sel;
  a.k = f.prof;
  a.piv = (const R*)f.piv;
  return a;
}

template <typename R>
size_t small_fdm_lds(const SmallFdm<R>& a, int N, bool stage) {
  size_t n = (size_t)3 * 16 * a.t1 * a.ld + 16 * a.t1;
  if (stage) n += (size_t)512 * (a.t0 * a.t0 + (a.line ? 0 : a.t1 * a.t1));
  return n * sizeof(R) + (size_t)(N + 3) / 4 * 4 * sizeof(double);
}

}  // namespace

template <typename R>
bool small_pcg_use(const piso_ctx* c) {
  if (c->dim != 2 || !c->fdm.on || c->N > kSmallCells || c->timing.enabled) return false;
  const SmallFdm<R> a = small_fdm<R>(c);
  return std::max(a.t0, a.line ? 0 : a.t1) <= kSmallTiles && small_fdm_lds<R>(a, c->N, false) <= kSmallLds;
}

template <typename R>
int small_pcg(piso_ctx* c, hipStream_t s, const R* Pf, const R* b, const double* mean, double sign, const R* x0, R* x,
              bool gauge, double tol2, double met2, int max_iter) {
  const SmallFdm<R> a = small_fdm<R>(c);
  const unsigned long long seq = ++c->wait_seq;
  const bool stage = small_fdm_lds<R>(a, c->N, true) <= kSmallLds;
  const size_t lds = small_fdm_lds<R>(a, c->N, stage);
  const int wg = small_threads(c->N, kPcgWG), cpt = (c->N + wg - 1) / wg;
#define SMALL_PCG(CPT, STAGE)                                                                                     \
  k_pcg_small<R, CPT, STAGE><<<1, wg, lds, s>>>(c->grid, a, Pf, b, mean, sign, x0, x, gauge ? 1 : 0, tol2, met2, \
                                                max_iter, c->cg, c->h_cg, seq)
#define SMALL_PCG_C(CPT)             \
  do {                               \
    if (stage) SMALL_PCG(CPT, true); \
    else SMALL_PCG(CPT, false);      \
  } while (0)
  if (cpt == 1) SMALL_PCG_C(1);
  else if (cpt == 2) SMALL_PCG_C(2);
  else SMALL_PCG_C(4);
#undef SMALL_PCG
#undef SMALL_PCG_C
  return small_check(c, s, &c->h_cg->seq, "k_pcg_small");
}

bool small_bi_use(const piso_ctx* c) {
  if (c->timing.enabled || c->cg_grid != 0) return false;   // as the pressure solve
  return c->N <= (c->dim == 3 ? 4 * kBiWG : kSmallCells);   // what the registers hold
}

template <typename R>
int small_bicgstab(piso_ctx* c, hipStream_t s, bool trans, const R* A, const R* C, const R* b, R* x, bool from_zero,
                   BiState* st, double tol2, int max_iter) {
  const unsigned long long seq = ++c->wait_seq;
  const size_t lds = (size_t)c->dim * c->N * sizeof(double);
  const int wg = small_threads(c->N, kBiWG), cpt = (c->N + wg - 1) / wg;
#define SMALL_BI(D, T, CPT) \
  k_bi_small<R, D, T, CPT><<<1, wg, lds, s>>>(c->grid, A, C, b, x, from_zero ? 1 : 0, st, c->h_bi, seq, tol2, \
                                              max_iter)
#define SMALL_BI_C(D, T)                  \
  do {                                    \
    if (cpt == 1) SMALL_BI(D, T, 1);      \
    else if (cpt == 2) SMALL_BI(D, T, 2); \
    else if (cpt <= 4) SMALL_BI(D, T, 4); \
    else if constexpr (D == 2) SMALL_BI(D, T, 8); \
  } while (0)
  if (c->dim == 2) {
    if (trans) SMALL_BI_C(2, true);
    else SMALL_BI_C(2, false);
  } else {
    if (trans) SMALL_BI_C(3, true);
    else SMALL_BI_C(3, false);
  }
#undef SMALL_BI
#undef SMALL_BI_C
  return small_check(c, s, &c->h_bi->seq, "k_bi_small");
}

#define INST(R)                                                                                                    \
  template bool small_pcg_use<R>(const piso_ctx*);                                                                 \
  template int small_pcg<R>(piso_ctx*, hipStream_t, const R*, const R*, const double*, double, const R*, R*, bool, \
                            double, double, int);                                                                  \
  template int small_bicgstab<R>(piso_ctx*, hipStream_t, bool, const R*, const R*, const R*, R*, bool, BiState*,    \
                                 double, int);
INST(float)
INST(double)
#undef INST

}  // namespace piso
