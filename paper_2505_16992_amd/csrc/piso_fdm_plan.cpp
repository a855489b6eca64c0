#include "piso_fdm_plan.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <numeric>
#include <thread>

namespace piso {

// Implicit-shift QR on a symmetric tridiagonal matrix (Golub and Van Loan, Matrix
// Computations, section 8.3): bulge chasing with Wilkinson's shift, the rotations applied
// to rows of the transposed vector matrix so that they run over contiguous memory.
bool tridiag_eigen(std::vector<double> a, std::vector<double> b, std::vector<double>* w, std::vector<double>* z) {
  const int n = (int)a.size();
  std::vector<double> zt((size_t)n * n, 0.0);   // row k: vector k
  for (int k = 0; k < n; ++k) zt[(size_t)k * n + k] = 1.0;
  const double eps = 2.3e-16;
  int hi = n - 1;
  long budget = 60L * n;
  while (hi > 0) {
    int lo = hi;
    while (lo > 0 && std::fabs(b[lo - 1]) > eps * (std::fabs(a[lo - 1]) + std::fabs(a[lo]))) --lo;
    if (lo > 0) b[lo - 1] = 0.0;
    if (lo == hi) {
      --hi;
      continue;
    }
    if (--budget < 0) return false;
    const double h = 0.5 * (a[hi - 1] - a[hi]), c2 = b[hi - 1] * b[hi - 1];
    const double mu = a[hi] - c2 / (h + (h >= 0 ? 1.0 : -1.0) * std::sqrt(h * h + c2));
    double x = a[lo] - mu, y = b[lo];
    for (int k = lo; k < hi; ++k) {
      const double r = std::hypot(x, y);
      const double c = r > 0 ? x / r : 1.0, s = r > 0 ? y / r : 0.0;
      if (k > lo) b[k - 1] = r;
      const double ak = a[k], bk = b[k], an = a[k + 1];
      a[k] = c * c * ak + 2.0 * c * s * bk + s * s * an;
      a[k + 1] = s * s * ak - 2.0 * c * s * bk + c * c * an;
      b[k] = c * s * (an - ak) + (c * c - s * s) * bk;
      if (k + 1 < hi) {
        x = b[k];
        y = s * b[k + 1];
        b[k + 1] *= c;
      }
      double* p = &zt[(size_t)k * n];
      double* q = p + n;
      for (int i = 0; i < n; ++i) {
        const double u = p[i], v = q[i];
        p[i] = c * u + s * v;
        q[i] = c * v - s * u;
      }
    }
  }
  std::vector<int> order(n);
  std::iota(order.begin(), order.end(), 0);
  std::sort(order.begin(), order.end(), [&](int p, int q) { return a[p] < a[q]; });
  w->resize(n);
  z->resize((size_t)n * n);
  for (int k = 0; k < n; ++k) {
    (*w)[k] = a[order[k]];
    for (int i = 0; i < n; ++i) (*z)[(size_t)i * n + k] = zt[(size_t)order[k] * n + i];
  }
  return true;
}

namespace {

// A matrix that its reversal leaves unchanged (an axis stretched the same way to both walls)
// of even size: even and odd vectors apart, two problems of half the size, a quarter of the
// work (n = 256: 19 against 5 ms).  False for any other.
bool mirror_eigen(const std::vector<double>& a, const std::vector<double>& b, std::vector<double>* w,
                  std::vector<double>* z) {
  const int n = (int)a.size(), h = n / 2;
  if (n % 2 || n < 4) return false;
  double scale = 0.0, off = 0.0;
  for (int i = 0; i < n; ++i) {
    scale = std::max(scale, std::fabs(a[i]));
    off = std::max(off, std::fabs(a[i] - a[n - 1 - i]));
    if (i + 1 < n) off = std::max(off, std::fabs(b[i] - b[n - 2 - i]));
  }
  if (!(off <= 1e-13 * scale)) return false;
  std::vector<double> wh[2], zh[2];
  for (int odd = 0; odd < 2; ++odd) {
    std::vector<double> ah(a.begin(), a.begin() + h), bh(b.begin(), b.begin() + h - 1);
    ah[h - 1] += odd ? -b[h - 1] : b[h - 1];
    if (!tridiag_eigen(ah, bh, &wh[odd], &zh[odd])) return false;
  }
  w->resize(n);
  z->resize((size_t)n * n);
  const double s = std::sqrt(0.5);
  for (int k = 0, p[2] = {0, 0}; k < n; ++k) {   // ascending
    const int odd = p[0] == h || (p[1] < h && wh[1][p[1]] < wh[0][p[0]]) ? 1 : 0;
    const int c = p[odd]++;
    (*w)[k] = wh[odd][c];
    for (int i = 0; i < h; ++i) {
      const double v = s * zh[odd][(size_t)i * h + c];
      (*z)[(size_t)i * n + k] = v;
      (*z)[(size_t)(n - 1 - i) * n + k] = odd ? -v : v;
    }
  }
  return true;
}

// One axis, one rung: K from the cell factors kf (face weights their mean), weights D.
bool axis_basis(const std::vector<double>& kf, const std::vector<double>& D, bool wrap, double* lam, double* V) {
  const int n = (int)kf.size();
  if (wrap) {   // the real Fourier basis (kf and D constant)
    const double pi = 3.14159265358979323846;
    for (int k = 0; k < n; ++k) {
      const int f = (k + 1) / 2;   // frequencies 0, 1, 1, 2, 2, ...: cosines at odd k, sines at even
      lam[k] = 2.0 * kf[0] / D[0] * (1.0 - std::cos(2.0 * pi * f / n));
      const bool plain = k == 0 || 2 * f == n;
      const double s = std::sqrt((plain ? 1.0 : 2.0) / (n * D[0]));
      for (int i = 0; i < n; ++i) {
        const double t = 2.0 * pi * (double)((long)f * i % n) / n;
        V[(size_t)i * n + k] = s * (k % 2 == 1 || k == 0 ? std::cos(t) : std::sin(t));
      }
    }
  } else {
    std::vector<double> a(n, 0.0), b(n > 1 ? n - 1 : 0), w, z;
    for (int i = 0; i + 1 < n; ++i) {
      const double f = 0.5 * (kf[i] + kf[i + 1]);
      a[i] += f;
      a[i + 1] += f;
      b[i] = -f / std::sqrt(D[i] * D[i + 1]);
    }
    for (int i = 0; i < n; ++i) a[i] /= D[i];
    if (!mirror_eigen(a, b, &w, &z) && !tridiag_eigen(a, b, &w, &z)) return false;
    for (int k = 0; k < n; ++k) {
      lam[k] = w[k];
      for (int i = 0; i < n; ++i) V[(size_t)i * n + k] = z[(size_t)i * n + k] / std::sqrt(D[i]);
    }
    double sum = 0.0;   // the null vector is the constant, exactly
    for (int i = 0; i < n; ++i) sum += D[i];
    for (int i = 0; i < n; ++i) V[(size_t)i * n] = 1.0 / std::sqrt(sum);
  }
  lam[0] = 0.0;
  for (int k = 1; k < n; ++k)
    if (!(lam[k] > 0.0) || !std::isfinite(lam[k])) return false;
  return true;
}

// Places the blocks on the lattice of a box: extents, periodic axes and the cell of every
// position.  False where they do not tile one, or a face is not where the box has it.
bool logical_box(const piso_domain_desc* d, const Topology& topo, int n[3], bool wrap[3], std::vector<int>* cell) {
  const int D = d->dim, B = d->n_blocks;
  const int* tab = topo.tab.data();
  auto ext = [&](int b, int m) { return tab[(size_t)b * kTabStride + 1 + m]; };
  std::vector<int> off(3 * (size_t)B, 0), todo(1, 0);
  std::vector<char> placed(B, 0);
  int period[3] = {0, 0, 0};
  placed[0] = 1;
  while (!todo.empty()) {
    const int b = todo.back();
    todo.pop_back();
    for (int s = 0; s < d->n_sides; ++s) {
      const piso_side_desc& sd = d->sides[s];
      if (sd.block != b || sd.kind != PISO_SIDE_CONNECT) continue;
      const int o = sd.other_block, a = sd.side / 2;
      int at[3], q = 0;
      for (int m = 0; m < 3; ++m) {
        at[m] = off[3 * b + m];
        if (m != a && q < 2) {
          at[m] += sd.begin[q] - sd.other_begin[q];
          ++q;
        }
      }
      at[a] += sd.side % 2 ? ext(b, a) : -ext(o, a);
      if (!placed[o]) {
        for (int m = 0; m < 3; ++m) off[3 * o + m] = at[m];
        placed[o] = 1;
        todo.push_back(o);
        continue;
      }
      // a second way to a block: a period along one axis
      int axis = -1, moved = 0;
      for (int m = 0; m < 3; ++m)
        if (at[m] != off[3 * o + m]) {
          axis = m;
          ++moved;
        }
      if (moved == 0) continue;
      const int len = std::abs(at[axis] - off[3 * o + axis]);
      if (moved > 1 || (period[axis] && period[axis] != len)) return false;
      period[axis] = len;
    }
  }
  for (int b = 0; b < B; ++b)
    if (!placed[b]) return false;
  long total = 1;
  int lo[3];
  for (int m = 0; m < 3; ++m) {
    int hi = off[m] + ext(0, m);
    lo[m] = off[m];
    for (int b = 1; b < B; ++b) {
      lo[m] = std::min(lo[m], off[3 * b + m]);
      hi = std::max(hi, off[3 * b + m] + ext(b, m));
    }
    wrap[m] = period[m] > 0;
    n[m] = wrap[m] ? period[m] : hi - lo[m];
    if (n[m] < 1 || n[m] > topo.N) return false;
    total *= n[m];
    if (total > topo.N) return false;
  }
  if (total != topo.N) return false;
  cell->assign(topo.N, -1);
  std::vector<int> where(topo.N);   // position of each cell
  for (int b = 0; b < B; ++b) {
    int P = tab[(size_t)b * kTabStride];
    for (int k = 0; k < ext(b, 2); ++k)
      for (int j = 0; j < ext(b, 1); ++j)
        for (int i = 0; i < ext(b, 0); ++i, ++P) {
          const int x[3] = {off[3 * b] - lo[0] + i, off[3 * b + 1] - lo[1] + j, off[3 * b + 2] - lo[2] + k};
          const int L = x[0] % n[0] + n[0] * (x[1] % n[1] + n[1] * (x[2] % n[2]));
          if ((*cell)[L] >= 0) return false;
          (*cell)[L] = P;
          where[P] = L;
        }
  }
  // every face of every block's side
  const int st[3] = {1, n[0], n[0] * n[1]};
  for (int b = 0; b < B; ++b)
    for (int side = 0; side < 2 * D; ++side) {
      const int* t = tab + (size_t)b * kTabStride;
      const int a = side / 2, hi = side % 2;
      int o[2], q = 0;
      for (int m = 0; m < 3; ++m)
        if (m != a && q < 2) o[q++] = m;
      const int bs[3] = {1, ext(b, 0), ext(b, 0) * ext(b, 1)};
      for (int v = 0, f = 0; v < ext(b, o[1]); ++v)
        for (int u = 0; u < ext(b, o[0]); ++u, ++f) {
          const int P = t[0] + (hi ? ext(b, a) - 1 : 0) * bs[a] + u * bs[o[0]] + v * bs[o[1]];
          const int F = topo.fmap[(size_t)t[4 + side] + f];
          const int x = where[P] / st[a] % n[a], y = hi ? x + 1 : x - 1;
          if (F < 0) {
            if (wrap[a] || (y >= 0 && y < n[a])) return false;
          } else {
            if (!wrap[a] && (y < 0 || y >= n[a])) return false;
            if (where[F] != where[P] + ((y + n[a]) % n[a] - x) * st[a]) return false;
          }
        }
    }
  return true;
}

}  // namespace

void fdm_plan(const piso_domain_desc* d, const Topology& topo, FdmPlan* plan) {
  plan->on = false;
  const int D = d->dim, N = topo.N;
  if (N < 2) return;
  int nb[3];
  bool wb[3];
  std::vector<int> box;
  if (!logical_box(d, topo, nb, wb, &box)) return;
  for (int m = 0; m < D; ++m)
    if (nb[m] > kFdmMaxN) return;
  plan->dim = D;
  // the line axis: y where it has walls, else z, else x (then x and y change places: the
  // line axis has to be strided in the box)
  const int walls = !wb[1] ? 1 : (D == 3 && !wb[2] ? 2 : (!wb[0] ? 0 : -1));
  if (walls == 0) std::swap(plan->perm[0], plan->perm[1]);
  const int la = plan->line = walls == 0 ? 1 : walls;
  int n[3], stride[3];
  for (int m = 0; m < 3; ++m) {
    plan->n[m] = n[m] = nb[plan->perm[m]];
    plan->wrap[m] = wb[plan->perm[m]];
  }
  stride[0] = 1;
  stride[1] = n[0];
  stride[2] = n[0] * n[1];
  if (walls == 0) {
    plan->cell.resize(N);
    for (int k = 0, L = 0; k < n[2]; ++k)
      for (int j = 0; j < n[1]; ++j)
        for (int i = 0; i < n[0]; ++i, ++L) plan->cell[L] = box[j + nb[0] * (i + nb[1] * k)];
  } else {
    plan->cell.swap(box);
  }
  plan->plain = true;
  for (int L = 0; L < N && plan->plain; ++L) plan->plain = plan->cell[L] == L;
  // alpha_jj by box axis and position
  auto alpha = [&](int j, int L) {
    const size_t P = plan->cell[L];
    const double* T = d->T + (size_t)plan->perm[j] * D * N + P;
    double s = 0.0;
    for (int i = 0; i < D; ++i) s += T[(size_t)i * N] * T[(size_t)i * N];
    return d->J[P] * s;
  };
  // up to 24 points of every axis (3D: 12, a plane still has 144), both ends' neighbourhoods
  // among them
  std::vector<int> pick[3];
  for (int m = 0; m < 3; ++m) {
    const int c = std::min(n[m], D == 3 ? 12 : 24);
    for (int u = 0; u < c; ++u) pick[m].push_back((int)((2L * u + 1) * n[m] / (2 * c)));
  }
  // f[j][m]: factor of alpha_jj along m, cj its scale (means of the logarithm); g[m]: the
  // faces of axis m in the diagonal of the diffusion (walls: 2 alpha), per volume
  std::vector<double> f[3][3], g[3];
  double cj[3] = {1, 1, 1}, gmax = 0.0;
  bool shape = false;
  for (int m = 0; m < D; ++m) {
    const int o0 = m == 0 ? 1 : 0, o1 = m == 2 ? 1 : 2;
    const std::vector<int> one(1, 0);
    const std::vector<int>&p0 = pick[o0], &p1 = D == 3 ? pick[o1] : one;
    const double cnt = (double)p0.size() * p1.size();
    g[m].assign(n[m], 0.0);
    for (int j = 0; j < D; ++j) f[j][m].assign(n[m], 0.0);
    for (int i = 0; i < n[m]; ++i)
      for (int u : p0)
        for (int v : p1) {
          const int L = i * stride[m] + u * stride[o0] + (D == 3 ? v * stride[o1] : 0);
          for (int j = 0; j < D; ++j) f[j][m][i] += std::log(alpha(j, L)) / cnt;
          const double own = alpha(m, L);
          double s = 0.0;
          for (int sd = -1; sd <= 1; sd += 2) {
            int r = i + sd;
            if (plan->wrap[m]) r = (r + n[m]) % n[m];
            s += r < 0 || r >= n[m] ? 2.0 * own : 0.5 * (own + alpha(m, L + (r - i) * stride[m]));
          }
          g[m][i] += s / d->J[plan->cell[L]] / cnt;
        }
    double lo = g[m][0], hi = g[m][0];
    for (double v : g[m]) {
      lo = std::min(lo, v);
      hi = std::max(hi, v);
    }
    gmax += hi;
    if (m != la && !plan->wrap[m] && hi > 1.05 * lo) shape = true;
    for (int j = 0; j < D; ++j) {
      double mean = 0.0;
      for (double v : f[j][m]) mean += v / n[m];
      if (m == 0) cj[j] = std::exp(mean);
      for (double& v : f[j][m]) {
        v = plan->wrap[m] && m != la ? 1.0 : std::exp(v - mean);   // Fourier basis: constant factors
        if (!(v > 0.0) || !std::isfinite(v)) return;
      }
      if (!(cj[j] > 0.0) || !std::isfinite(cj[j])) return;
    }
  }
  if (!std::isfinite(gmax)) return;
  // weights of an axis with a basis: one for all other directions' terms
  std::vector<double> w[3];
  for (int m = 0; m < D; ++m) {
    w[m].assign(n[m], 1.0);
    for (int i = 0; i < n[m]; ++i) {
      double l = 0.0;
      for (int j = 0; j < D; ++j)
        if (j != m) l += std::log(f[j][m][i]) / (D - 1);
      w[m][i] = std::exp(l);
    }
  }
  // spread of the metric's face weights about the product, relative to the plane means
  {
    const int pa = la >= 0 ? la : 1;
    const int cells = N / n[pa];
    std::vector<double> v(3 * (size_t)n[pa] * 3, 0.0);   // [plane][term][min, max, sum]
    for (int q = 0; q < 3 * n[pa]; ++q) v[3 * (size_t)q] = HUGE_VAL;
    const int oa = pa == 1 ? 2 : 1;
    auto planes = [&](int beg, int end) {
      for (int pl = beg; pl < end; ++pl)
        for (int o = 0; o < n[oa]; ++o)
          for (int i = 0; i < n[0]; ++i) {
            int x[3] = {i, 0, 0};
            x[pa] = pl;
            x[oa] = o;
            const int L = i + x[1] * stride[1] + x[2] * stride[2];
            double* pv = &v[(size_t)pl * 9];
            for (int j = 0; j < D; ++j) {
              double m0 = cj[j];
              for (int m = 0; m < D; ++m)
                if (m != la) m0 *= m == j ? f[m][m][x[m]] : w[m][x[m]];
              const double r = alpha(j, L) / m0;
              pv[3 * j] = std::min(pv[3 * j], r);
              pv[3 * j + 1] = std::max(pv[3 * j + 1], r);
              pv[3 * j + 2] += r / cells;
            }
          }
    };
    // large grids in threads (96^3: 23 ms on one core); a thread that cannot start runs here
    const int T = std::min(n[pa], N > 100000 ? 8 : 1);
    std::vector<std::thread> pool;
    pool.reserve(T);
    for (int t = 0; t < T; ++t) {
      const int beg = (int)((long)n[pa] * t / T), end = (int)((long)n[pa] * (t + 1) / T);
      if (t + 1 == T) {
        planes(beg, end);
        continue;
      }
      try {
        pool.emplace_back(planes, beg, end);
      } catch (...) {   // std::system_error, or std::bad_alloc for the thread itself
        planes(beg, end);
      }
    }
    for (std::thread& th : pool) th.join();
    double lo = HUGE_VAL, hi = 0.0;
    for (int pl = 0; pl < n[pa]; ++pl)
      for (int j = 0; j < D; ++j) {
        const double* pv = &v[(size_t)pl * 9 + 3 * j];
        const double mean = la >= 0 ? pv[2] : 1.0;
        lo = std::min(lo, pv[0] / mean);
        hi = std::max(hi, pv[1] / mean);
      }
    if (!(hi <= kFdmMaxShape * lo) || !(lo > 0.0)) return;
  }
  plan->rungs = shape ? kFdmRungs : 1;
  const int Q = plan->rungs;
  for (int m = 0; m < D; ++m) {
    if (m != la) {
      plan->lam[m].assign((size_t)Q * n[m], 0.0);
      plan->V[m].assign((size_t)Q * n[m] * n[m], 0.0);
    }
    for (int j = 0; j < D; ++j) plan->wt[j][m].assign((size_t)Q * n[m], 1.0);
  }
  struct Job {
    int m, q;
    std::vector<double> kf, D;
    bool ok;
  };
  std::vector<Job> jobs;
  for (int q = 0; q < Q; ++q) {
    const double s = kFdmLadder[q] / gmax;
    for (int m = 0; m < D; ++m) {
      if (m == la) continue;
      // a_m: mean of log 1 / (1 + s g) over the other axes
      std::vector<double> a(n[m], 1.0);
      if (s > 0.0 && !plan->wrap[m]) {
        const int o0 = m == 0 ? 1 : 0, o1 = m == 2 ? 1 : 2;
        double mean = 0.0;
        for (int i = 0; i < n[m]; ++i) {
          double l = 0.0;
          for (int u : pick[o0])
            for (int v : pick[o1]) l -= std::log(1.0 + s * (g[m][i] + g[o0][u] + (D == 3 ? g[o1][v] : 0.0)));
          a[i] = l / ((double)pick[o0].size() * pick[o1].size());
          mean += a[i] / n[m];
        }
        for (double& v : a) v = std::exp(v - mean);
      }
      Job job{m, q, std::vector<double>(n[m]), std::vector<double>(n[m]), false};
      for (int i = 0; i < n[m]; ++i) {
        job.kf[i] = cj[m] * f[m][m][i] * a[i];
        job.D[i] = w[m][i] * a[i];
        for (int j = 0; j < D; ++j) plan->wt[j][m][(size_t)q * n[m] + i] = job.D[i];
      }
      for (int i = 0; i < n[m]; ++i) {
        const int r = i + 1 < n[m] ? i + 1 : 0;
        plan->wt[m][m][(size_t)q * n[m] + i] = 0.5 * (job.kf[i] + job.kf[r]);
      }
      jobs.push_back(std::move(job));
    }
  }
  auto build = [&](Job& b) {
    const int nm = plan->n[b.m];
    try {
      b.ok = axis_basis(b.kf, b.D, plan->wrap[b.m], &plan->lam[b.m][(size_t)b.q * nm],
                        &plan->V[b.m][(size_t)b.q * nm * nm]);
    } catch (...) {
      b.ok = false;
    }
  };
  // long axes in threads (n = 256: about 30 ms a basis); a thread that cannot start runs here
  std::vector<std::thread> pool;
  pool.reserve(jobs.size());
  for (Job& b : jobs) {
    if (b.kf.size() < 64 || plan->wrap[b.m]) {
      build(b);
      continue;
    }
    try {
      pool.emplace_back(build, std::ref(b));
    } catch (...) {
      build(b);
    }
  }
  for (std::thread& th : pool) th.join();
  for (const Job& b : jobs)
    if (!b.ok) return;
  plan->on = true;
}

}  // namespace piso
