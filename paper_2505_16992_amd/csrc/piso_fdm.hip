// Fast-diagonalisation preconditioner of the pressure PCG on blocks that form a logical box
// with a metric near a tensor product (plan and mathematics: piso_fdm_plan.h).  z = B r with
// one dense product per axis and direction, and one tridiagonal system per mode along the line
// axis: GEMM-shaped work on fields of N cells, done with the FP32 / FP64 matrix instructions
// (full precision of the type, no narrower operands).
//
// What bounds it.  2 n flops per cell and product over two field streams: at n = 96 in FP32
// that is 24 flop/B, about the ratio of the chip's 150 TFLOP/s of FP32 matrix rate to its
// 5 TB/s, and a pass over a 96^3 field is a few microseconds either way, where the launch
// counts as much.  So every product reads its operand once into LDS and the small basis
// from the L2, and products are fused with what stands next to them:
//   k_fdm_row, MODE 1   PCG update (alpha, x, r') and the forward product along x
//   k_fdm_col, MODE 0   forward product along the remaining axis (3D)
//   k_fdm_line          the tridiagonal systems; without a line axis (y and z periodic)
//                       k_fdm_col, MODE 2: forward product, 1 / Lambda, inverse product
//   k_fdm_col, MODE 1   inverse product along the remaining axis (3D)
//   k_fdm_row, MODE 2   inverse product along x and the partial sums of r.z, r.r
// An iteration is these and the stencil kernel: 4 launches in 2D and 6 in 3D, against 7 to
// 11 with the multigrid V-cycle, and it needs 2 to 25 iterations where the V-cycle needs
// 15 to 80 (the spectrum of B M lies within the spread of the ratios of the face weights of
// M and M0).
//
// Tiles.  Matrix instructions of 16 x 16 outputs: the basis is the A operand, packed on the
// host so that a lane's four consecutive k are one 16- or 32-byte load; the field tile is
// the B operand, from LDS.  The order of k is the same in both, so any order will do: lane
// group g takes k = k0 + 4 g + t for the t-th of four instructions.  A wave owns 16-row
// output tiles over all columns of the work-group's field tile; where a field has too few
// tiles to fill the chip (2D), several work-groups share a field tile and split its output
// rows (`splits`).
//
// Transformed fields are in box order.  Where that is not the cells' order (several blocks,
// x and y exchanged) the two products along x, which meet the cells, go through a map.
//
// The constant mode.  M has it for its null space and the residual's sum is zero, but in FP32
// the sum left by rounding is enough to stop the iteration from reaching 1e-7 (a 105 x 171
// cavity went from 2e-7 to 1 and stayed there).  The kernel that meets the null mode knows
// the residual's mean exactly; it leaves it in device memory, and the next kernels that read
// the residual take it off (no pass of its own).
//
// Per operator (once a step for both correctors): k_fdm_stats and k_fdm_select compare its
// face weights with each rung's, keep the plane means as the line systems' profiles and the
// rung of the smallest spread in device memory (no read-back); a spread above kFdmMaxSpread
// marks the operator as rejected, k_cg_check ends the solve before its first iteration and
// the host runs it with multigrid.  k_fdm_factor then forms the pivots.
#include <algorithm>
#include <cstdlib>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "piso_fdm_plan.h"
#include "piso_impl.h"
#include "piso_mma.h"

namespace piso {

namespace {

constexpr int kFdmMaxWaves = 8;
constexpr int kFdmPad = 4;   // LDS row padding: the 16 rows (row tiles) or the four k groups
                             // (column tiles) of an operand read fall on different banks

}  // namespace

// ------------------------------------------------------------------- products along x

template <typename R>
struct FdmRow {
  int n, rows, kc, mt, splits, mper, ks, ntiles, ld;   // mper: output tiles per split, ks: waves sharing one
  uint32_t div_lo, div_hi;                         // division by n (or n / 4)
  int div_sh, quad;
  const int* map;
  int rowfast;
  const R* V;
  size_t vstride;
  const FdmSel* sel;   // rung and the mean of r
  const R* in;         // MODE 0: r; MODE 1: r (before the update); MODE 2: transformed field
  R* out;
  R *x, *rout;         // MODE 1
  const R *dnew, *q;
  const R* r;          // MODE 2: residual for the partial sums
  CgState* st;
  const double* partA;
  double* partB;
  int Gp, par;
};

// Sum of G partials, the same in every thread of every work-group of the launch.
__device__ __forceinline__ double fdm_partials(const double* __restrict__ part, int G, double* red) {
  double v = 0.0;
  for (int w0 = 0; w0 < G; w0 += 8 * (int)blockDim.x) {
    double u[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int w = w0 + (int)threadIdx.x + c * (int)blockDim.x;
      u[c] = w < G ? part[w] : 0.0;
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) v += u[c];
  }
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < (int)blockDim.x >> 6; ++w) t += red[w];
  __syncthreads();
  return t;
}

// GATHER (MODE 0 and 1): cells one by one, through the map or on rows that are no quads; a form
// of its own, since its eight loads in flight cost the quad form registers (96^3: 9.5 us
// alone, 12.0 with both in one kernel).
template <typename R, int NT, int MODE, bool GATHER>
__global__ void __launch_bounds__(64 * kFdmMaxWaves) k_fdm_row(FdmRow<R> a) {
  using V4 = typename Vec4<R>::T;
  extern __shared__ __align__(32) char smem[];
  __shared__ double red[2 * kFdmMaxWaves];
  R* X = (R*)smem;   // [16 NT][ld]
  const int done = a.st->done;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nth = blockDim.x;
  const int g = lane >> 4, nl = lane & 15;
  const uint64_t dm = (uint64_t)a.div_lo | ((uint64_t)a.div_hi << 32);
  const bool qin = a.quad && !GATHER;
  const int per_row = qin ? a.n >> 2 : a.n;
  const int total = a.ntiles * a.splits;
  R alpha = R(0);
  if constexpr (MODE == 1) {
    const double rzp = a.st->rz[a.par];
    const double dq = fdm_partials(a.partA, a.Gp, red);
    if (done) return;
    if (!(dq > 0.0) || !std::isfinite(dq)) {
      if (blockIdx.x == 0 && tid == 0) {
        a.st->status = std::isfinite(dq) ? PISO_BREAKDOWN : PISO_E_NAN;
        a.st->iters = a.st->k;
        a.st->done = 1;
      }
      return;
    }
    alpha = (R)(rzp / dq);
    if (blockIdx.x == 0 && tid == 0) a.st->k = a.st->k + 1;   // no other work-group reads it here
  } else {
    if (done) return;
  }
  const R* Vq = a.V + (size_t)a.sel->q * a.vstride;
  const R mean = MODE == 0 ? R(0) : (R)a.sel->mean;
  double acc_rz = 0.0, acc_rr = 0.0;
  for (int lt = xcd_logical_group(); lt < total; lt += gridDim.x) {
    const int tile = lt / a.splits, sp = lt % a.splits;
    const int row0 = tile * 16 * NT;
    const int rows = min(16 * NT, a.rows - row0);
    const size_t base = (size_t)row0 * a.n;
    // field tile into LDS (without a map contiguous in memory); the first split also stores
    // the update
    // (eight elements' loads at a time: through the map each is two loads in a row, and one by
    // one a 256 x 256 grid took 12.5 us here)
    auto gather = [&](int count, auto&& at) {
      constexpr int U = 8;
      for (int e0 = tid; e0 < count; e0 += U * nth) {
        int rr[U], cc[U];
        size_t P[U];
        R v[U], qv[U], xv[U], dv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int e = min(e0 + u * nth, count - 1);
          P[u] = at(e, rr[u], cc[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          v[u] = a.in[P[u]];
          if constexpr (MODE == 1) {
            qv[u] = a.q[P[u]];
            if (sp == 0) {
              xv[u] = a.x[P[u]];
              dv[u] = a.dnew[P[u]];
            }
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (e0 + u * nth >= count || rr[u] >= rows) continue;
          if constexpr (MODE == 1) {
            v[u] = (v[u] - mean) - alpha * qv[u];
            if (sp == 0) {
              a.x[P[u]] = xv[u] + alpha * dv[u];
              a.rout[P[u]] = v[u];
            }
          }
          X[rr[u] * a.ld + cc[u]] = v[u];
        }
      }
    };
    if constexpr (GATHER) {
      if (a.rowfast)
        gather(16 * NT * a.n, [&](int e, int& r, int& c) {
          r = e % (16 * NT);
          c = e / (16 * NT);
          return (size_t)a.map[(size_t)c * a.rows + row0 + min(r, rows - 1)];
        });
      else
        gather(rows * per_row, [&](int e, int& r, int& c) {
          r = (int)fast_div((uint32_t)e, dm, a.div_sh);
          c = e - r * per_row;
          return a.map ? (size_t)a.map[base + e] : base + e;
        });
    } else {
      for (int e = tid; e < rows * per_row; e += nth) {
        const int r = (int)fast_div((uint32_t)e, dm, a.div_sh);
        if (MODE == 2 && !qin) {   // the transformed field is in box order
          X[r * a.ld + (e - r * per_row)] = a.in[base + e];
          continue;
        }
        const int c = (e - r * per_row) << 2;
        const size_t P = base + (size_t)e * 4;
        V4 v = *reinterpret_cast<const V4*>(a.in + P);
        if constexpr (MODE == 1) {
          const V4 qv = *reinterpret_cast<const V4*>(a.q + P);
          const bool own = sp == 0;
          V4 xv, dv;
          if (own) {
            xv = *reinterpret_cast<const V4*>(a.x + P);
            dv = *reinterpret_cast<const V4*>(a.dnew + P);
          }
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = (v[t] - mean) - alpha * qv[t];
          if (own) {
#pragma unroll
            for (int t = 0; t < 4; ++t) xv[t] += alpha * dv[t];
            *reinterpret_cast<V4*>(a.x + P) = xv;
            *reinterpret_cast<V4*>(a.rout + P) = v;
          }
        }
        R* d = X + r * a.ld + c;
#pragma unroll
        for (int t = 0; t < 4; ++t) d[t] = v[t];
      }
    }
    // zeros beyond the row's end and in missing rows (the packed basis is zero there too, but
    // stale LDS may hold NaN)
    const int tail = a.kc * 16 - a.n;
    for (int e = tid; e < 16 * NT * tail; e += nth) X[(e / tail) * a.ld + a.n + e % tail] = R(0);
    for (int e = tid; e < (16 * NT - rows) * a.n; e += nth) X[(rows + e / a.n) * a.ld + e % a.n] = R(0);
    __syncthreads();
    const int mend = min(a.mt, (sp + 1) * a.mper);
    // with ks > 1 each wave has one output tile and a part of its sum (mper * ks waves)
    const int wk = wave % a.ks, wm = wave / a.ks, k0 = a.kc * wk / a.ks, k1 = a.kc * (wk + 1) / a.ks;
    for (int m = wm; m < a.mper; m += (nth >> 6) / a.ks) {
      const int mt = sp * a.mper + m;
      V4 acc[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = V4{R(0), R(0), R(0), R(0)};
      if (mt < mend) {
        const R* vp = Vq + ((size_t)mt * a.kc * 64 + lane) * 4;
#pragma unroll 4
        for (int k = k0; k < k1; ++k) {
          const V4 av = *reinterpret_cast<const V4*>(vp + (size_t)k * 256);
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const V4 bv = lds4<R>(X + (t * 16 + nl) * a.ld + k * 16 + 4 * g);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[t] = mma(av[u], bv[u], acc[t]);
          }
        }
      }
      if (a.ks > 1) {   // every wave is here once
        R* part = X + (size_t)16 * NT * a.ld + ((size_t)wm * a.ks * 64 + lane) * 4 * NT;
        if (wk > 0) {
#pragma unroll
          for (int t = 0; t < NT; ++t) sts4<R>(part + (size_t)wk * 256 * NT + 4 * t, acc[t]);
        }
        __syncthreads();
        if (wk > 0) continue;
        for (int w = 1; w < a.ks; ++w)
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[t] += lds4<R>(part + (size_t)w * 256 * NT + 4 * t);
      }
      if (mt >= mend) continue;
      const int col = mt * 16 + 4 * g;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int r = t * 16 + nl;
        if (r >= rows || col >= a.n) continue;
        const size_t P = base + (size_t)r * a.n + col;
        if (a.quad && (MODE != 2 || !a.map)) {
          *reinterpret_cast<V4*>(a.out + P) = acc[t];
          if constexpr (MODE == 2) {
            const V4 rv = *reinterpret_cast<const V4*>(a.r + P);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const double rp = (double)(rv[u] - mean);
              acc_rz += rp * (double)acc[t][u];
              acc_rr += rp * rp;
            }
          }
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (col + u >= a.n) continue;
            size_t Q = P + u;
            if (MODE == 2 && a.map) Q = a.map[a.rowfast ? (size_t)(col + u) * a.rows + row0 + r : Q];
            a.out[Q] = acc[t][u];
            if constexpr (MODE == 2) {
              const double rp = (double)(a.r[Q] - mean);
              acc_rz += rp * (double)acc[t][u];
              acc_rr += rp * rp;
            }
          }
        }
      }
    }
    __syncthreads();   // before the next tile overwrites X
  }
  if constexpr (MODE == 2) {
    const double s0 = wave_sum(acc_rz), s1 = wave_sum(acc_rr);
    if (lane == 0) {
      red[wave] = s0;
      red[kFdmMaxWaves + wave] = s1;
    }
    __syncthreads();
    if (tid == 0) {
      double t0 = 0.0, t1 = 0.0;
      for (int w = 0; w < nth >> 6; ++w) {
        t0 += red[w];
        t1 += red[kFdmMaxWaves + w];
      }
      a.partB[blockIdx.x] = t0;
      a.partB[gridDim.x + blockIdx.x] = t1;
    }
  }
}

// --------------------------------------------------------------- products along y or z

template <typename R>
struct FdmCol {
  int n, kc, mt, splits, mper, ld;
  int cols, ctiles;      // contiguous columns of one slab, tiles per slab
  int slabs;
  size_t sstride, rstride;   // cells between slabs, between rows
  int quad;
  const R *Vf, *Vi;
  size_t vstride;
  const R *lr, *lc, *ls;     // eigenvalues along the rows, the columns, the slabs (or null)
  const double* ones;
  FdmSel* sel;
  const R* in;
  R* out;
  const CgState* st;
};

// MODE 0: forward; 1: inverse; 2: forward, 1 / Lambda, inverse; 3: forward, 1 / Lambda.
template <typename R, int NT, int MODE>
__global__ void __launch_bounds__(64 * kFdmMaxWaves) k_fdm_col(FdmCol<R> a) {
  using V4 = typename Vec4<R>::T;
  constexpr int TN = 16 * NT;
  extern __shared__ __align__(32) char smem[];
  R* X = (R*)smem;                       // [16 kc][ld]
  R* Y = X + (size_t)a.kc * 16 * a.ld;   // MODE 2: [16 kc][ld]
  if (a.st->done) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nth = blockDim.x;
  const int g = lane >> 4, nl = lane & 15;
  const int lt = xcd_logical_group();
  const int sp = lt % a.splits, tile = lt / a.splits;
  const int slab = tile / a.ctiles, c0 = (tile - slab * a.ctiles) * TN;
  const size_t base = (size_t)slab * a.sstride + c0;
  const int q = a.sel->q;
  if (a.quad) {
    for (int e = tid; e < a.kc * 16 * (TN / 4); e += nth) {
      const int r = e / (TN / 4), c = (e % (TN / 4)) * 4;
      V4 v = V4{R(0), R(0), R(0), R(0)};
      if (r < a.n && c0 + c < a.cols) v = *reinterpret_cast<const V4*>(a.in + base + (size_t)r * a.rstride + c);
      R* d = X + r * a.ld + c;
#pragma unroll
      for (int t = 0; t < 4; ++t) d[t] = v[t];
    }
  } else {
    for (int e = tid; e < a.kc * 16 * TN; e += nth) {
      const int r = e / TN, c = e % TN;
      X[r * a.ld + c] = r < a.n && c0 + c < a.cols ? a.in[base + (size_t)r * a.rstride + c] : R(0);
    }
  }
  __syncthreads();
  const R* Vq = (MODE == 1 ? a.Vi : a.Vf) + (size_t)q * a.vstride;
  R lcol[NT] = {};
  if constexpr (MODE >= 2) {
    const R ls = a.ls ? a.ls[(size_t)q * a.slabs + slab] : R(0);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int c = c0 + t * 16 + nl;
      lcol[t] = ls + a.lc[(size_t)q * a.cols + (c < a.cols ? c : 0)];
    }
  }
  const R* src = X;
#pragma unroll
  for (int pass = 0; pass < (MODE == 2 ? 2 : 1); ++pass) {
    const int mend = min(a.mt, (sp + 1) * a.mper);
    for (int mt = sp * a.mper + wave; mt < mend; mt += nth >> 6) {
      V4 acc[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = V4{R(0), R(0), R(0), R(0)};
      const R* vp = Vq + ((size_t)mt * a.kc * 64 + lane) * 4;
#pragma unroll 4
      for (int k = 0; k < a.kc; ++k) {
        const V4 av = *reinterpret_cast<const V4*>(vp + (size_t)k * 256);
        const R* xs = src + (size_t)(k * 16 + 4 * g) * a.ld + nl;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[t] = mma(av[u], xs[u * a.ld + t * 16], acc[t]);
      }
      const int row = mt * 16 + 4 * g;
      if constexpr (MODE >= 2) {
        if (pass == 0) {
          if (slab == 0 && c0 == 0 && mt == 0 && lane == 0) a.sel->mean = (double)acc[0][0] * a.ones[q];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const R lr = row + u < a.n ? a.lr[(size_t)q * a.n + row + u] : R(0);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              const R l = lr + lcol[t];
              acc[t][u] = row + u < a.n && l > R(0) ? acc[t][u] / l : R(0);   // the null mode is left out
            }
          }
        }
      }
      if (MODE == 2 && pass == 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int t = 0; t < NT; ++t) Y[(row + u) * a.ld + t * 16 + nl] = acc[t][u];
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (row + u >= a.n) continue;
          R* o = a.out + base + (size_t)(row + u) * a.rstride;
#pragma unroll
          for (int t = 0; t < NT; ++t)
            if (c0 + t * 16 + nl < a.cols) o[t * 16 + nl] = acc[t][u];
        }
      }
    }
    if (MODE == 2 && pass == 0) {
      __syncthreads();
      src = Y;
      Vq = a.Vi + (size_t)q * a.vstride;
    }
  }
}

// ------------------------------------------------------------ tridiagonal line systems

// Per mode (c, slab) of the other two axes the rows of [K + diag(lc c_x + ls c_s)] w = h, K
// the stiffness of the couplings k.  Factorised from both ends to the middle row m = n / 2
// (two lanes a column, half the chain of dependent steps), every step a sum of positive
// terms: with e the row's excess over its open coupling,
//   top:    e_j = q_j + k_{j-1} e_{j-1} / p_{j-1},  p_j = k_j + e_j
//   bottom: e_j = q_j + k_j e_{j+1} / p_{j+1},      p_j = k_{j-1} + e_j
//   middle: p_m = q_m + both neighbours' terms,
// so that the smallest pivots (smooth modes) keep their relative accuracy in FP32 fields.
// The null mode (q = 0) is pinned at the middle row; its right-hand side and its solution are
// freed of their means.
template <typename R>
struct FdmLine {
  int n, cols, slabs;
  size_t sstride, rstride;
  const R *lc, *ls;      // [rung][cols], [rung][slabs] (or null)
  const double *k, *cx, *cs;   // profiles along the line: couplings, weights of lc and of ls
  const double* ones;
  FdmSel* sel;
  R* piv;
  const R* in;
  R* out;
  const CgState* st;
};

template <typename R>
__global__ void __launch_bounds__(64) k_fdm_factor(FdmLine<R> a) {
  if (a.sel->bad) return;
  const int lane = threadIdx.x, half = lane >> 5;
  const int per = (a.cols + 31) / 32;
  const int slab = blockIdx.x / per, c0 = (blockIdx.x - slab * per) * 32 + (lane & 31);
  const bool on = c0 < a.cols;
  const int c = on ? c0 : a.cols - 1;
  const int q = a.sel->q, n = a.n, m = n / 2;
  const double lx = (double)a.lc[(size_t)q * a.cols + c];
  const double ls = a.ls ? (double)a.ls[(size_t)q * a.slabs + slab] : 0.0;
  R* piv = a.piv + (size_t)slab * a.sstride + c;
  auto diag = [&](int j) { return lx * a.cx[j] + (a.ls ? ls * a.cs[j] : 0.0); };
  // rows 0 .. m - 1 downward (half 0), n - 1 .. m + 1 upward (half 1); eight rows' profile
  // loads at a time, ahead of the chain
  const int steps = half ? n - 1 - m : m;
  double carry = 0.0;   // k e / p of the row before
  constexpr int B = 8;
  for (int t0 = 0; t0 < steps; t0 += B) {
    double open[B], dg[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int t = min(t0 + u, steps - 1), j = half ? n - 1 - t : t;
      open[u] = a.k[half ? j - 1 : j];
      dg[u] = diag(j);
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if (t0 + u >= steps) break;
      const int j = half ? n - 1 - (t0 + u) : t0 + u;
      const double e = dg[u] + carry;
      const double ip = 1.0 / (open[u] + e);
      carry = open[u] * e * ip;
      if (on) piv[(size_t)j * a.rstride] = (R)ip;
    }
  }
  const double other = __shfl_xor(carry, 32, 64);
  if (half == 0 && on) {
    double p = diag(m) + (carry + other);
    if (!(p > 0.0)) p = n > 1 ? (m > 0 ? a.k[m - 1] : 0.0) + (m + 1 < n ? a.k[m] : 0.0) : 0.0;
    piv[(size_t)m * a.rstride] = p > 0.0 ? (R)(1.0 / p) : R(0);
  }
}

// The solve.  With y = value / pivot the recurrences are one FMA a row,
//   forward  y_j = r_j I_j + (k_before I_j) y_before,   backward  x_j = y_j + (k_after I_j) x_after
// (I: reciprocal pivots), and all three coefficients are formed by the whole work-group while
// it brings a tile of TN columns to LDS.  What is left to the one wave that runs the chains is
// then issue-bound: rows lie contiguous per column in the order the chain meets them (the
// lower half reversed, zeros ahead of its first row up to a multiple of four), so that four
// rows are two 16-byte LDS reads, four FMAs and a write.  256 rows of 256 columns: 20 us with
// row-by-row addressing, of which the two chains took most, now 9.0.
__host__ __device__ inline int line_len(int n) { return (n / 2 + 3) / 4 * 4; }   // longer half, padded
// column stride: 4 modulo 8, so that the columns' 16-byte reads spread over the banks
__host__ __device__ inline int line_stride(int n) { return line_len(n) + (line_len(n) % 8 ? 8 : 4); }
template <typename R>
inline size_t line_lds(int n, int tn) {
  return ((size_t)6 * tn * line_stride(n) + 4 * (size_t)tn) * sizeof(R);
}

template <typename R, int TN>
__global__ void __launch_bounds__(kWG) k_fdm_line(FdmLine<R> a) {
  using V4 = typename Vec4<R>::T;
  extern __shared__ __align__(32) char smem[];
  __shared__ double red[kWaves];
  const int n = a.n, m = n / 2, Lp = line_len(n), L = line_stride(n), T = 2 * TN * L;
  R* Y = (R*)smem;     // [half][column][L]: r I, then y, then the solution
  R* G = Y + T;        // k_before I
  R* F = G + T;        // k_after I
  R* Rm = F + T;       // [TN] middle row's r I, then its solution
  R* Mc = Rm + TN;     // [half][TN] middle row's k I towards each half
  if (a.st->done) return;
  const int tid = threadIdx.x;
  const int per = (a.cols + TN - 1) / TN;
  const int tile = xcd_logical_group(), slab = tile / per, c0 = (tile - slab * per) * TN;
  const size_t base = (size_t)slab * a.sstride + c0;
  const int w = min(TN, a.cols - c0);
  // the null mode is column 0 of the first tile: its right-hand side's mean
  const bool null = slab == 0 && c0 == 0;
  R off = R(0);
  auto block_sum = [&](double t) {
    t = wave_sum(t);
    if ((tid & 63) == 0) red[tid >> 6] = t;
    __syncthreads();
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) v += red[q];
    __syncthreads();
    return v;
  };
  if (null) {
    double t = 0.0;
    for (int j = tid; j < n; j += kWG) t += (double)a.in[(size_t)j * a.rstride];
    t = block_sum(t);
    off = (R)(t / n);
    if (tid == 0) a.sel->mean = t * a.ones[a.sel->q];
  }
  constexpr int U = 8;
  for (int e0 = tid; e0 < n * TN; e0 += U * kWG) {
    R xv[U], iv[U], kb[U], ka[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kWG, j = min(e / TN, n - 1), c = e % TN;
      const size_t P = c < w ? base + (size_t)j * a.rstride + c : base;
      xv[u] = a.in[P];
      iv[u] = a.piv[P];
      kb[u] = (R)a.k[max(j - 1, 0)];
      ka[u] = (R)a.k[j];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * kWG, j = e / TN, c = e % TN;
      if (j >= n) continue;
      const R x = c == 0 ? xv[u] - off : xv[u];
      const R lo = j > 0 ? kb[u] * iv[u] : R(0), hi = j + 1 < n ? ka[u] * iv[u] : R(0);
      if (j == m) {
        Rm[c] = x * iv[u];
        Mc[c] = lo;
        Mc[TN + c] = hi;
      } else {
        const int half = j > m, steps = half ? n - 1 - m : m, t = half ? n - 1 - j : j;
        const int q = (half * TN + c) * L + Lp - steps + t;
        Y[q] = x * iv[u];
        G[q] = half ? hi : lo;
        F[q] = half ? lo : hi;
      }
    }
  }
  for (int e = tid; e < 2 * TN * 4; e += kWG) {   // zeros ahead of a half's first row
    const int half = e / (TN * 4), c = e / 4 % TN, p = e % 4;
    if (p < Lp - (half ? n - 1 - m : m)) {
      const int q = (half * TN + c) * L + p;
      Y[q] = G[q] = F[q] = R(0);
    }
  }
  __syncthreads();
  if (tid < 2 * TN) {
    const int half = tid / TN, c = tid % TN;
    R *y = Y + (half * TN + c) * L, *g = G + (half * TN + c) * L, *f = F + (half * TN + c) * L;
    R d = R(0);
    V4 yv = lds4<R>(y), gv = lds4<R>(g);
    for (int p = 0; p < Lp; p += 4) {
      const V4 yn = lds4<R>(y + p + 4), gn = lds4<R>(g + p + 4);   // the padding behind the last
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        d = yv[u] + gv[u] * d;
        yv[u] = d;
      }
      sts4<R>(y + p, yv);
      yv = yn;
      gv = gn;
    }
    const R mine = Mc[half * TN + c] * d;
    const R other = __shfl_xor(mine, TN, 64);
    R x = Rm[c] + (half ? other + mine : mine + other);
    if (half == 0) Rm[c] = x;
    if (Lp > 0) {
      V4 ya = lds4<R>(y + Lp - 4), fa = lds4<R>(f + Lp - 4);
      for (int p = Lp - 4; p >= 0; p -= 4) {
        const int pn = max(p - 4, 0);
        const V4 yn = lds4<R>(y + pn), fn = lds4<R>(f + pn);
#pragma unroll
        for (int u = 3; u >= 0; --u) {
          x = ya[u] + fa[u] * x;
          ya[u] = x;
        }
        sts4<R>(y + p, ya);
        ya = yn;
        fa = fn;
      }
    }
  }
  __syncthreads();
  auto value = [&](int j, int c) {
    const int half = j > m, steps = half ? n - 1 - m : m, t = half ? n - 1 - j : j;
    return j == m ? Rm[c] : Y[(half * TN + c) * L + Lp - steps + t];
  };
  R shift = R(0);   // the null mode's solution without its mean
  if (null) {
    double t = 0.0;
    for (int j = tid; j < n; j += kWG) t += (double)value(j, 0);
    shift = (R)(block_sum(t) / n);
  }
  for (int e = tid; e < n * TN; e += kWG) {
    const int j = e / TN, c = e % TN;
    if (c < w) a.out[base + (size_t)j * a.rstride + c] = value(j, c) - (c == 0 ? shift : R(0));
  }
}

// ------------------------------------------------------ profiles and choice of a rung

template <typename R>
struct FdmStats {
  int dim, rungs, pa, oa, splits;   // planes normal to pa; oa: the other axis of their rows
  int n[3], wrap[3], perm[3];
  size_t stride[3];
  size_t N;
  const int* map;
  int rowfast;
  const R* wt[3][3];   // [j][m]: [rung][n_m], reciprocals of the weights' factors
};
constexpr int kFdmMaxSplits = 4;        // work-groups a plane
constexpr int kFdmStatValues = 3 * 3;   // per rung: term, then smallest, largest, sum

// Smallest, largest and sum of the ratios of the operator's face weights to each rung's over
// the planes normal to pa, `splits` work-groups a plane.  A weight that is not positive or
// not finite gives an infinite spread.  One read of P_f, once per operator.
template <typename R>
__global__ void __launch_bounds__(kWG) k_fdm_stats(FdmStats<R> a, const R* __restrict__ Pf, float* __restrict__ out) {
  __shared__ float sh[kFdmRungs * kFdmStatValues][kWaves];
  float lo[kFdmRungs][3], hi[kFdmRungs][3], sum[kFdmRungs][3];
#pragma unroll
  for (int q = 0; q < kFdmRungs; ++q)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      lo[q][j] = INFINITY;
      hi[q][j] = sum[q][j] = 0.f;
    }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lg = xcd_logical_group(), plane = lg / a.splits, sp = lg % a.splits;
  const int nx = a.n[0], segs = (nx + 63) / 64, rows = a.n[a.oa];
  constexpr int U = 4;   // row segments whose loads are in flight together
  const int step = a.splits * kWaves;
  for (int w0 = sp * kWaves + wave; w0 < rows * segs; w0 += U * step) {
    R p[U][3];
    int oo[U], ii[U];
    bool on[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int w = min(w0 + u * step, rows * segs - 1);
      oo[u] = w / segs;
      ii[u] = (w - oo[u] * segs) * 64 + lane;
      on[u] = w0 + u * step < rows * segs && ii[u] < nx;
      const int i = min(ii[u], nx - 1);
      size_t P = (size_t)plane * a.stride[a.pa] + (size_t)oo[u] * a.stride[a.oa] + i;
      if (a.map) P = a.map[a.rowfast ? (size_t)i * (a.N / nx) + P / nx : P];
#pragma unroll
      for (int j = 0; j < 3; ++j) p[u][j] = j < a.dim ? Pf[(size_t)a.perm[j] * a.N + P] : R(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!on[u]) continue;
      const int i = ii[u], o = oo[u];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (j >= a.dim) continue;
        const int pos = j == 0 ? i : (j == a.pa ? plane : o);
        if (pos + 1 >= a.n[j] && !a.wrap[j]) continue;
#pragma unroll
        for (int q = 0; q < kFdmRungs; ++q) {
          if (q >= a.rungs) continue;
          R m = a.wt[j][0][q * nx + i] * a.wt[j][a.pa][q * a.n[a.pa] + plane];   // 1 / weight
          if (a.dim == 3) m *= a.wt[j][a.oa][q * rows + o];
          const float v = (float)(p[u][j] * m);
          const bool ok = v > 0.f && std::isfinite(v);
          lo[q][j] = ok ? fminf(lo[q][j], v) : 0.f;
          hi[q][j] = ok ? fmaxf(hi[q][j], v) : INFINITY;
          sum[q][j] += v;
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kFdmRungs; ++q)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      if (q >= a.rungs) continue;
#pragma unroll
      for (int s = 32; s > 0; s >>= 1) {
        lo[q][j] = fminf(lo[q][j], __shfl_xor(lo[q][j], s, 64));
        hi[q][j] = fmaxf(hi[q][j], __shfl_xor(hi[q][j], s, 64));
        sum[q][j] += __shfl_xor(sum[q][j], s, 64);
      }
      if (lane == 0) {
        float(*v)[kWaves] = &sh[q * kFdmStatValues + 3 * j];
        v[0][wave] = lo[q][j];
        v[1][wave] = hi[q][j];
        v[2][wave] = sum[q][j];
      }
    }
  __syncthreads();
  const int v = threadIdx.x;
  if (v < a.rungs * kFdmStatValues) {
    float t = sh[v][0];
    for (int w = 1; w < kWaves; ++w) t = v % 3 == 0 ? fminf(t, sh[v][w]) : (v % 3 == 1 ? fmaxf(t, sh[v][w]) : t + sh[v][w]);
    out[(size_t)v * gridDim.x + lg] = t;
  }
}

// Rung of the smallest spread over all faces (relative to the plane means along a line axis),
// and the means as that rung's profiles: prof[0] couplings along the line, prof[1] weights of
// the x term, prof[2] weights of the third term.  One work-group, a wave per rung, every load
// of a plane's statistics in flight at once (one rung after the other, load by load, six rungs
// took 13 - 14 us; now 5 - 7).
constexpr int kFdmSelectWG = 512;
static_assert(kFdmRungs <= kFdmSelectWG / 64, "a wave per rung");
__global__ void __launch_bounds__(kFdmSelectWG)
k_fdm_select(const float* __restrict__ st, int planes, int splits, int rungs, int dim, int pa, int line,
             int3 faces, int last_open, float limit, double* __restrict__ prof, FdmSel* sel, CgState* host,
             unsigned long long seq) {
  __shared__ float spread[kFdmRungs];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const size_t G = (size_t)planes * splits;
  constexpr int S = kFdmMaxSplits;
  // the three statistics of direction j on plane pl
  auto stat = [&](int rung, int j, int pl, float (&v)[3]) {
    float t[3][S];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int s = 0; s < S; ++s)
        t[k][s] = st[(size_t)(rung * kFdmStatValues + 3 * j + k) * G + (size_t)pl * splits + min(s, splits - 1)];
    v[0] = t[0][0];
    v[1] = t[1][0];
    v[2] = t[2][0];
#pragma unroll
    for (int s = 1; s < S; ++s) {   // a repeated split changes neither extreme
      v[0] = fminf(v[0], t[0][s]);
      v[1] = fmaxf(v[1], t[1][s]);
      v[2] += s < splits ? t[2][s] : 0.f;
    }
  };
  auto count = [&](int j, int pl) {
    if (j == pa && last_open && pl + 1 == planes) return 0;
    return j == 0 ? faces.x : (j == 1 ? faces.y : faces.z);
  };
  if (q < rungs) {
    float lo = INFINITY, hi = 0.f;
    for (int pl = lane; pl < planes; pl += 64) {
      float v[3][3];
#pragma unroll
      for (int j = 0; j < 3; ++j) stat(q, min(j, dim - 1), pl, v[j]);
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int cnt = j < dim ? count(j, pl) : 0;
        if (cnt == 0) continue;
        const float mean = line ? v[j][2] / (float)cnt : 1.f;
        const float l = v[j][0] / mean, h = v[j][1] / mean;
        lo = l > 0.f ? fminf(lo, l) : 0.f;     // also 0 where the mean is infinite or NaN
        hi = h > 0.f ? fmaxf(hi, h) : INFINITY;
      }
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
      lo = fminf(lo, __shfl_xor(lo, s, 64));
      hi = fmaxf(hi, __shfl_xor(hi, s, 64));
    }
    if (lane == 0) spread[q] = lo > 0.f ? hi / lo : INFINITY;
  }
  __syncthreads();
  float top = INFINITY;
  int best = 0;
  for (int k = 0; k < rungs; ++k)
    if (spread[k] < top) {
      top = spread[k];
      best = k;
    }
  if (threadIdx.x == 0) {
    sel->q = best;
    sel->bad = top <= limit ? 0 : 1;
    if (host) {   // pinned
      host->status = top <= limit ? 0 : kFdmRejected;
      publish(&host->seq, seq);
    }
  }
  if (!line) return;
  for (int e = threadIdx.x; e < planes * dim; e += kFdmSelectWG) {
    const int j = e / planes, pl = e - j * planes, cnt = count(j, pl);
    float v[3];
    stat(best, j, pl, v);
    const int slot = j == pa ? 0 : (j == 0 ? 1 : 2);
    prof[(size_t)slot * planes + pl] = cnt ? (double)v[2] / cnt : 0.0;
  }
}

// ------------------------------------------------------------------------- host side

namespace {

// V (or its transpose) of every rung in operand order, zero-padded to multiples of 16.  Read in
// memory order, each element to its place: lane 16 (k / 4) + (place of the output row), step
// k % 4 of its 16 x 16 block.
template <typename R>
std::vector<R> pack(const FdmPlan& p, int m, bool fwd) {
  const int n = p.n[m], T = (n + 15) / 16;
  std::vector<R> out((size_t)p.rungs * T * T * 256, R(0));
  int place[16];
  for (int l = 0; l < 16; ++l) place[packed_row<R>(l)] = l;
  const double* v = p.V[m].data();
  for (int q = 0; q < p.rungs; ++q)
    for (int row = 0; row < n; ++row)
      for (int col = 0; col < n; ++col, ++v) {
        const int k = fwd ? row : col, o = fwd ? col : row;
        const size_t block = ((size_t)q * T + o / 16) * T + k / 16;
        out[(block * 64 + 16 * (k % 16 / 4) + place[o % 16]) * 4 + k % 4] = (R)*v;
      }
  return out;
}

template <typename R>
std::vector<R> narrow(const std::vector<double>& v) {
  return std::vector<R>(v.begin(), v.end());
}

std::vector<double> reciprocal(std::vector<double> v) {
  for (double& x : v) x = 1.0 / x;
  return v;
}

template <typename R>
int upload_plan(piso_ctx* c, const FdmPlan& p) {
  FdmState& f = c->fdm;
  for (int m = 0; m < p.dim; ++m) {
    if (m != p.line) {
      if (int rc = upload(c, &f.fwd[m], pack<R>(p, m, true))) return rc;
      if (int rc = upload(c, &f.inv[m], pack<R>(p, m, false))) return rc;
      if (int rc = upload(c, &f.lam[m], narrow<R>(p.lam[m]))) return rc;
    }
    for (int j = 0; j < p.dim; ++j)
      if (int rc = upload(c, &f.wt[j][m], narrow<R>(reciprocal(p.wt[j][m])))) return rc;
  }
  std::vector<double> ones(p.rungs, 1.0 / c->N);
  for (int m = 0; m < p.dim; ++m)
    for (int q = 0; q < p.rungs && m != p.line; ++q) ones[q] /= p.V[m][(size_t)q * p.n[m] * p.n[m]];
  if (int rc = upload(c, (void**)&f.ones, ones)) return rc;
  if (p.line >= 0)
    if (int rc = dev_alloc(c, &f.piv, (size_t)c->N * sizeof(R))) return rc;
  return dev_alloc(c, &f.hat, (size_t)c->N * sizeof(R));
}

// Columns per field tile (16 NT), work-groups sharing a tile and waves per work-group for an
// axis of mt output tiles and `units` columns or rows.  Wide tiles reuse a basis operand for
// several instructions; narrow ones and splits keep about two work-groups per CU in flight.
struct Shape {
  int nt, splits, mper, waves, ks;
};
Shape shape_for(long units, int mt, int max_nt, bool may_split) {
  Shape s;
  s.nt = 1;
  while (s.nt < max_nt && units / (16L * s.nt * 2) >= 512) s.nt *= 2;
  const long tiles = (units + 16L * s.nt - 1) / (16L * s.nt);
  s.splits = 1;
  if (may_split)
    while (tiles * s.splits < 256 && (mt + 2 * s.splits - 1) / (2 * s.splits) >= 2) s.splits *= 2;
  s.mper = (mt + s.splits - 1) / s.splits;
  s.splits = (mt + s.mper - 1) / s.mper;
  // as many waves as divide the output tiles evenly, at least 4 for the loads
  const int trips = (s.mper + kFdmMaxWaves - 1) / kFdmMaxWaves;
  s.waves = std::max(4, (s.mper + trips - 1) / trips);
  s.ks = 1;
  return s;
}

// LDS of a column tile; MODE 2 holds two
template <typename R>
size_t col_lds(int n, int nt, bool fused) {
  return (size_t)((n + 15) / 16 * 16) * (16 * nt + kFdmPad) * sizeof(R) * (fused ? 2 : 1);
}
constexpr size_t kFdmLds = 150 * 1024;

template <typename R, int MODE>
void launch_row(piso_ctx* c, hipStream_t s, int kind, FdmRow<R> a, const Shape& sh, int G) {
  const bool gather = MODE != 2 && (!a.quad || a.map);
  const bool qin = a.quad && !gather;   // as in the kernel
  div_magic((uint32_t)(qin ? a.n / 4 : a.n), a.div_lo, a.div_hi, a.div_sh);
  const size_t lds = ((size_t)16 * sh.nt * a.ld + (sh.ks > 1 ? (size_t)sh.waves * 256 * sh.nt : 0)) * sizeof(R);
  const int wg = 64 * sh.waves;
  auto launch = [&](auto nt) {
    constexpr int NT = decltype(nt)::value;
    if constexpr (MODE != 2) {
      if (gather) {
        launch_timed_lds(c, s, kind, k_fdm_row<R, NT, MODE, true>, G, wg, lds, a);
        return;
      }
    }
    launch_timed_lds(c, s, kind, k_fdm_row<R, NT, MODE, false>, G, wg, lds, a);
  };
  if (sh.nt == 1) launch(std::integral_constant<int, 1>{});
  else if (sh.nt == 2) launch(std::integral_constant<int, 2>{});
  else launch(std::integral_constant<int, 4>{});
}

template <typename R, int MODE>
void launch_col(piso_ctx* c, hipStream_t s, FdmCol<R> a, const Shape& sh) {
  a.ld = 16 * sh.nt + kFdmPad;
  a.splits = sh.splits;
  a.mper = sh.mper;
  a.ctiles = (a.cols + 16 * sh.nt - 1) / (16 * sh.nt);
  const size_t lds = col_lds<R>(a.n, sh.nt, MODE == 2);
  const int G = a.slabs * a.ctiles * a.splits, wg = 64 * sh.waves;
  if (sh.nt == 1) launch_timed_lds(c, s, kTimeMgCoarse, k_fdm_col<R, 1, MODE>, G, wg, lds, a);
  else if (sh.nt == 2) launch_timed_lds(c, s, kTimeMgCoarse, k_fdm_col<R, 2, MODE>, G, wg, lds, a);
  else launch_timed_lds(c, s, kTimeMgCoarse, k_fdm_col<R, 4, MODE>, G, wg, lds, a);
}

template <typename R>
Shape row_shape(const piso_ctx* c) {
  const int nx = c->fdm.n[0];
  const int max_nt = nx * sizeof(R) <= 1024 ? 4 : 2;   // tile within half the LDS
  const int kc = (nx + 15) / 16;
  Shape s = shape_for((long)c->N / nx, kc, max_nt, true);
  // output rows split over work-groups leave one or two tiles to each: its waves then share a
  // tile's sum, at least two 16-cell chunks each (256^2 FP32: 6.7 us for the update and 6.5 for
  // the inverse with one of four waves at work on 16 chunks, 5.6 with eight on two each)
  if (s.splits > 1) {
    int ks = 1;
    while (2 * ks * s.mper <= kFdmMaxWaves && kc >= 4 * ks) ks *= 2;
    if (ks > 1) {
      s.ks = ks;
      s.waves = s.mper * ks;
    }
  }
  return s;
}

template <typename R>
int row_tiles(const piso_ctx* c, const Shape& sh) {
  const int rows = c->N / c->fdm.n[0];
  return (rows + 16 * sh.nt - 1) / (16 * sh.nt) * sh.splits;
}

int fdm_check(piso_ctx* c) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(c, PISO_E_HIP, std::string("k_fdm: ") + hipGetErrorString(e));
  return PISO_OK;
}

template <typename R>
FdmRow<R> row_args(piso_ctx* c, const Shape& sh, CgState* st) {
  const FdmState& f = c->fdm;
  FdmRow<R> a{};
  a.n = f.n[0];
  a.rows = c->N / a.n;
  a.kc = a.mt = (a.n + 15) / 16;
  a.splits = sh.splits;
  a.mper = sh.mper;
  a.ks = sh.ks;
  a.ntiles = (a.rows + 16 * sh.nt - 1) / (16 * sh.nt);
  a.ld = a.kc * 16 + kFdmPad;
  a.quad = a.n % 4 == 0;
  a.map = f.map;
  a.rowfast = f.rowfast;
  a.vstride = (size_t)a.mt * a.kc * 256;
  a.sel = f.sel;
  a.st = st;
  return a;
}

// Arguments of the line kernels: columns along x, slabs along the remaining axis.
template <typename R>
FdmLine<R> line_args(piso_ctx* c) {
  const FdmState& f = c->fdm;
  const bool d3 = c->dim == 3;
  const int la = f.line, oa = la == 1 ? 2 : 1;
  FdmLine<R> a{};
  a.n = f.n[la];
  a.cols = f.n[0];
  a.slabs = f.n[oa];   // 1 in 2D
  a.rstride = la == 1 ? f.n[0] : (size_t)f.n[0] * f.n[1];
  a.sstride = la == 1 ? (size_t)f.n[0] * f.n[1] : f.n[0];
  a.lc = (const R*)f.lam[0];
  a.ls = d3 ? (const R*)f.lam[oa] : nullptr;
  a.ones = f.ones;
  a.k = f.prof;
  a.cx = f.prof + f.planes;
  a.cs = f.prof + 2 * (size_t)f.planes;
  a.sel = f.sel;
  a.piv = (R*)f.piv;
  return a;
}

// 32 columns a tile (whole 128-byte lines in FP32), fewer where the chip would not fill or two
// tiles of the line do not fit the LDS
template <typename R>
int line_cols(const FdmLine<R>& a) {
  for (int tn : {32, 16}) {
    const bool fits = line_lds<R>(a.n, tn) <= kFdmLds;
    if (fits && (long)a.slabs * ((a.cols + tn - 1) / tn) >= 4 * tn) return tn;
  }
  return 8;
}

// The products and solves between the two products along x: transformed field in c->k_y,
// result in *res.
template <typename R>
int middle(piso_ctx* c, hipStream_t s, CgState* st, R** res) {
  const FdmState& f = c->fdm;
  const bool d3 = c->dim == 3;
  const int nx = f.n[0], ny = f.n[1], nz = f.n[2];
  R *u = (R*)c->k_y, *v = (R*)f.hat;
  FdmCol<R> a{};
  a.quad = nx % 4 == 0;
  a.sel = f.sel;
  a.st = st;
  auto along = [&](int m) {
    a.n = f.n[m];
    a.kc = a.mt = (a.n + 15) / 16;
    a.vstride = (size_t)a.mt * a.kc * 256;
    a.Vf = (const R*)f.fwd[m];
    a.Vi = (const R*)f.inv[m];
    a.rstride = m == 1 ? nx : (size_t)nx * ny;
    a.cols = m == 1 ? nx : nx * ny;
    a.slabs = m == 1 ? nz : 1;
    a.sstride = (size_t)nx * ny;
  };
  auto step = [&](auto mode, const Shape& sh) {
    a.in = u;
    a.out = v;
    launch_col<R, decltype(mode)::value>(c, s, a, sh);
    std::swap(u, v);
  };
  // 3D: the axis between x and the line (z, or y where the lines run along z)
  const int ma = f.line == 2 ? 1 : 2;
  Shape shm{};
  if (d3) {
    along(ma);
    const int max_nt =
        col_lds<R>(a.n, 4, false) <= kFdmLds / 2 ? 4 : (col_lds<R>(a.n, 2, false) <= kFdmLds / 2 ? 2 : 1);
    shm = shape_for((long)a.cols * a.slabs, a.mt, max_nt, true);
    step(std::integral_constant<int, 0>{}, shm);
  }
  if (f.line >= 0) {
    FdmLine<R> l = line_args<R>(c);
    l.in = u;
    l.out = v;
    l.st = st;
    const int tn = line_cols(l);
    const size_t lds = line_lds<R>(l.n, tn);
    const int G = l.slabs * ((l.cols + tn - 1) / tn);
    if (tn == 32) launch_timed_lds(c, s, kTimeMgCoarse, k_fdm_line<R, 32>, G, kWG, lds, l);
    else if (tn == 16) launch_timed_lds(c, s, kTimeMgCoarse, k_fdm_line<R, 16>, G, kWG, lds, l);
    else launch_timed_lds(c, s, kTimeMgCoarse, k_fdm_line<R, 8>, G, kWG, lds, l);
    std::swap(u, v);
  } else {
    along(1);
    a.lr = (const R*)f.lam[1];
    a.lc = (const R*)f.lam[0];
    a.ls = d3 ? (const R*)f.lam[2] : nullptr;
    a.ones = f.ones;
    // one kernel for both products and the scaling between them where its tiles fill the
    // chip (or the axis is short), else the output rows of each are split over work-groups:
    // a 2D 256^2 grid has 16 tiles of 16 columns
    const int max_nt = col_lds<R>(ny, 2, true) <= kFdmLds / 2 ? 2 : 1;
    const Shape shf = shape_for((long)nx * nz, a.mt, max_nt, false);
    const long tiles = (long)nz * ((nx + 16 * shf.nt - 1) / (16 * shf.nt));
    if (col_lds<R>(ny, shf.nt, true) <= kFdmLds && (tiles >= 96 || a.mt <= 4)) {
      step(std::integral_constant<int, 2>{}, shf);
    } else {
      const Shape sh = shape_for((long)nx * nz, a.mt, col_lds<R>(ny, 4, false) <= kFdmLds / 2 ? 4 : 1, true);
      step(std::integral_constant<int, 3>{}, sh);
      step(std::integral_constant<int, 1>{}, sh);
    }
  }
  if (d3) {
    along(ma);
    step(std::integral_constant<int, 1>{}, shm);
  }
  *res = u;
  return fdm_check(c);
}

template <typename R>
int finish(piso_ctx* c, hipStream_t s, const R* r, R* z, CgState* st, double* partB) {
  R* hat = nullptr;
  if (int rc = middle<R>(c, s, st, &hat)) return rc;
  const Shape sh = row_shape<R>(c);
  FdmRow<R> a = row_args<R>(c, sh, st);
  a.V = (const R*)c->fdm.inv[0];
  a.in = hat;
  a.out = z;
  a.r = r;
  a.partB = partB;
  launch_row<R, 2>(c, s, kTimeMgUp0, a, sh, fdm_groups<R>(c));
  return fdm_check(c);
}

}  // namespace

int fdm_build(piso_ctx* c, const piso_domain_desc* desc, const Topology& topo) {
  // a multigrid form asked for by name keeps the multigrid (PISO_MG_LINE and PISO_ZMARCH
  // choose its fine-level kernels)
  if (c->mg.empty() || std::getenv("PISO_MG_LINE") || std::getenv("PISO_ZMARCH")) return PISO_OK;
  if (c->dim == 3 && c->N < kFdmMinCells3) return PISO_OK;
  FdmPlan p;
  try {
    fdm_plan(desc, topo, &p);
    if (!p.on) return PISO_OK;
    FdmState& f = c->fdm;
    f.rungs = p.rungs;
    f.line = p.line;
    for (int m = 0; m < 3; ++m) {
      f.n[m] = p.n[m];
      f.wrap[m] = p.wrap[m];
      f.perm[m] = p.perm[m];
    }
    if (!p.plain) {
      f.rowfast = p.perm[0] != 0;
      if (f.rowfast) {
        const int nx = p.n[0], rows = c->N / nx;
        std::vector<int> t(c->N);
        for (int r = 0; r < rows; ++r)
          for (int i = 0; i < nx; ++i) t[(size_t)i * rows + r] = p.cell[(size_t)r * nx + i];
        p.cell.swap(t);
      }
      if (int rc = upload(c, (void**)&f.map, p.cell)) return rc;
    }
    if (int rc = c->prec == PISO_F64 ? upload_plan<double>(c, p) : upload_plan<float>(c, p)) return rc;
    // statistics: up to about 512 work-groups, at least a row segment per wave
    const int pa = f.line == 2 ? 2 : 1, oa = pa == 1 ? 2 : 1;
    f.planes = f.n[pa];
    const int units = f.n[oa] * ((f.n[0] + 63) / 64);
    f.splits = std::max(1, std::min({kFdmMaxSplits, 512 / f.planes, (units + kWaves - 1) / kWaves}));
    if (int rc = dev_alloc(c, (void**)&f.stats,
                           sizeof(float) * kFdmRungs * kFdmStatValues * (size_t)f.planes * f.splits))
      return rc;
    if (int rc = dev_alloc(c, (void**)&f.prof, sizeof(double) * 3 * (size_t)f.planes)) return rc;
    if (int rc = dev_alloc(c, (void**)&f.sel, sizeof(FdmSel))) return rc;
    PISO_HIP(c, hipMemset(f.sel, 0, sizeof(FdmSel)));
    f.on = true;
  } catch (const std::bad_alloc&) {
    return fail(c, PISO_E_OOM, "fast diagonalisation: host memory");
  }
  return PISO_OK;
}

template <typename R>
int fdm_groups(const piso_ctx* c) {
  return std::min(row_tiles<R>(c, row_shape<R>(c)), kRedGrid);
}

template <typename R>
int fdm_setup(piso_ctx* c, hipStream_t s, const R* Pf, bool wait) {
  const FdmState& f = c->fdm;
  FdmStats<R> a{};
  a.dim = c->dim;
  a.N = c->N;
  a.rungs = f.rungs;
  a.pa = f.line == 2 ? 2 : 1;
  a.oa = a.pa == 1 ? 2 : 1;
  a.splits = f.splits;
  a.stride[0] = 1;
  a.stride[1] = f.n[0];
  a.stride[2] = (size_t)f.n[0] * f.n[1];
  a.map = f.map;
  a.rowfast = f.rowfast;
  int3 faces;
  int* nf[3] = {&faces.x, &faces.y, &faces.z};
  for (int m = 0; m < 3; ++m) {
    a.n[m] = f.n[m];
    a.wrap[m] = f.wrap[m];
    a.perm[m] = f.perm[m];
    for (int j = 0; j < 3; ++j) a.wt[j][m] = (const R*)f.wt[j][m];
    const int cells = c->N / f.n[a.pa];   // of a plane
    *nf[m] = m == a.pa || f.wrap[m] ? cells : cells / f.n[m] * (f.n[m] - 1);
  }
  k_fdm_stats<R><<<f.planes * f.splits, kWG, 0, s>>>(a, Pf, f.stats);
  k_fdm_select<<<1, kFdmSelectWG, 0, s>>>(f.stats, f.planes, f.splits, f.rungs, c->dim, a.pa,
                                           f.line >= 0 ? 1 : 0, faces,
                                           f.wrap[a.pa] ? 0 : 1, kFdmMaxSpread, f.prof, f.sel,
                                           wait ? c->h_cg : nullptr, wait ? ++c->wait_seq : 0);
  if (wait) {
    if (int rc = fdm_check(c)) return rc;
    if (int rc = wait_pinned(c, s, &c->h_cg->seq, "k_fdm_select")) return rc;
    if (c->h_cg->status == kFdmRejected) return PISO_OK;
  }
  if (f.line >= 0) {
    const FdmLine<R> l = line_args<R>(c);
    k_fdm_factor<R><<<l.slabs * ((l.cols + 31) / 32), 64, 0, s>>>(l);
  }
  return fdm_check(c);
}

const int* fdm_rejected(const piso_ctx* c) { return &c->fdm.sel->bad; }

template <typename R>
int fdm_apply(piso_ctx* c, hipStream_t s, const R* r, R* z, CgState* st, double* partB) {
  const Shape sh = row_shape<R>(c);
  FdmRow<R> a = row_args<R>(c, sh, st);
  a.V = (const R*)c->fdm.fwd[0];
  a.in = r;
  a.out = (R*)c->k_y;
  launch_row<R, 0>(c, s, kTimeMgDown0, a, sh, row_tiles<R>(c, sh));
  return finish<R>(c, s, r, z, st, partB);
}

template <typename R>
int fdm_update_apply(piso_ctx* c, hipStream_t s, R* x, const R* rin, R* rout, const R* dnew, const R* q, R* z,
                     CgState* st, const double* partA, int Gp, int par, double* partB) {
  const Shape sh = row_shape<R>(c);
  FdmRow<R> a = row_args<R>(c, sh, st);
  a.V = (const R*)c->fdm.fwd[0];
  a.in = rin;
  a.out = (R*)c->k_y;
  a.x = x;
  a.rout = rout;
  a.dnew = dnew;
  a.q = q;
  a.partA = partA;
  a.Gp = Gp;
  a.par = par;
  launch_row<R, 1>(c, s, kTimeCgUpdateMg, a, sh, row_tiles<R>(c, sh));
  return finish<R>(c, s, (const R*)rout, z, st, partB);
}

#define INST(R)                                                                                                \
  template int fdm_groups<R>(const piso_ctx*);                                                                 \
  template int fdm_setup<R>(piso_ctx*, hipStream_t, const R*, bool);                                           \
  template int fdm_apply<R>(piso_ctx*, hipStream_t, const R*, R*, CgState*, double*);                          \
  template int fdm_update_apply<R>(piso_ctx*, hipStream_t, R*, const R*, R*, const R*, const R*, R*, CgState*, \
                                   const double*, int, int, double*);
INST(float)
INST(double)
#undef INST

}  // namespace piso
