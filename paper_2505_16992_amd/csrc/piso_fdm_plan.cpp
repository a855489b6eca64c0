#include "piso_fdm_plan.h"

#include <algorithm>
#include <cmath>
#include <numeric>
#include <system_error>
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

// One axis, one rung: K from the cell factors kf (face weights their mean), weights D.
bool axis_basis(const std::vector<double>& kf, const std::vector<double>& D, bool wrap, double* lam, double* V) {
  const int n = (int)kf.size();
  if (wrap) {   // uniform: the real Fourier basis
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
    if (!tridiag_eigen(a, b, &w, &z)) return false;
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

}  // namespace

void fdm_plan(const piso_domain_desc* d, const Topology& topo, FdmPlan* plan) {
  plan->on = false;
  const int D = d->dim, N = topo.N;
  if (d->n_blocks != 1 || N < 2) return;
  const int* t = topo.tab.data();
  int n[3], stride[3];
  for (int m = 0; m < 3; ++m) n[m] = t[1 + m];
  stride[0] = 1;
  stride[1] = n[0];
  stride[2] = n[0] * n[1];
  plan->dim = D;
  for (int m = 0; m < D; ++m) {
    if (n[m] > kFdmMaxN) return;
    const int w = (t[kTabWrap] >> (2 * m)) & 3;
    if (w == 1 || w == 2) return;
    plan->wrap[m] = w == 3;
    if (w == 0) {
      const int faces = N / n[m];
      for (int sd = 0; sd < 2; ++sd)
        for (int f = 0; f < faces; ++f)
          if (topo.fmap[(size_t)t[4 + 2 * m + sd] + f] >= 0) return;
    }
  }
  for (int m = 0; m < 3; ++m) plan->n[m] = n[m];
  // the line axis: y where it has walls, else z
  const int la = plan->line = !plan->wrap[1] ? 1 : (D == 3 && !plan->wrap[2] ? 2 : -1);
  // alpha_jj on the three mid-lines, then the test that it is their product everywhere
  auto alpha = [&](int j, size_t P) {
    double s = 0.0;
    for (int i = 0; i < D; ++i) {
      const double v = d->T[(size_t)(j * D + i) * N + P];
      s += v * v;
    }
    return d->J[P] * s;
  };
  size_t mid = 0;
  for (int m = 0; m < D; ++m) mid += (size_t)(n[m] / 2) * stride[m];
  std::vector<double> f[3][3], g[3];
  double cj[3] = {0, 0, 0};
  for (int j = 0; j < D; ++j) {
    cj[j] = alpha(j, mid);
    if (!(cj[j] > 0.0) || !std::isfinite(cj[j])) return;
    for (int m = 0; m < D; ++m) {
      f[j][m].resize(n[m]);
      for (int i = 0; i < n[m]; ++i) {
        f[j][m][i] = alpha(j, mid + ((long)i - n[m] / 2) * stride[m]) / cj[j];
        if (!(f[j][m][i] > 0.0) || !std::isfinite(f[j][m][i])) return;
      }
    }
  }
  // (a tolerance well above rounding: the basis only preconditions)
  const double tol = 1e-8;
  for (int k = 0, P = 0; k < n[2]; ++k)
    for (int jj = 0; jj < n[1]; ++jj) {
      double row[3];
      for (int j = 0; j < D; ++j) row[j] = cj[j] * f[j][1][jj] * (D == 3 ? f[j][2][k] : 1.0);
      for (int i = 0; i < n[0]; ++i, ++P)
        for (int j = 0; j < D; ++j) {
          const double v = row[j] * f[j][0][i];
          if (!(std::fabs(alpha(j, P) - v) <= tol * v)) return;
        }
    }
  // the weights of an axis with a basis have to be the same in every other direction's term
  for (int m = 0; m < D && D == 3; ++m) {
    if (m == la) continue;
    const int j0 = m == 0 ? 1 : 0, j1 = m == 2 ? 1 : 2;
    for (int i = 0; i < n[m]; ++i)
      if (!(std::fabs(f[j0][m][i] - f[j1][m][i]) <= tol * f[j0][m][i])) return;
  }
  // g_m(i): the faces of axis m in the diagonal of the diffusion (walls: 2 alpha), per volume
  double gmax = 0.0;
  bool shape = false;
  for (int m = 0; m < D; ++m) {
    g[m].resize(n[m]);
    double lo = 0.0, hi = 0.0;
    for (int i = 0; i < n[m]; ++i) {
      const double own = f[m][m][i];
      double s = 0.0;
      for (int sd = -1; sd <= 1; sd += 2) {
        int r = i + sd;
        if (plan->wrap[m]) r = (r + n[m]) % n[m];
        s += r < 0 || r >= n[m] ? 2.0 * own : 0.5 * (own + f[m][m][r]);
      }
      g[m][i] = cj[m] * s / d->J[mid + ((long)i - n[m] / 2) * stride[m]];
      lo = i ? std::min(lo, g[m][i]) : g[m][i];
      hi = std::max(hi, g[m][i]);
    }
    if (!std::isfinite(hi)) return;
    if (plan->wrap[m]) {   // Fourier basis: uniform axes only
      for (int i = 0; i < n[m]; ++i)
        for (int j = 0; j < D; ++j)
          if (!(std::fabs(f[j][m][i] - f[j][m][0]) <= tol * f[j][m][0])) return;
    } else if (m != la && hi > 1.05 * lo) {
      shape = true;
    }
    gmax += hi;
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
      // a_m: mean of log 1 / (1 + s g) over the other axes, up to 24 points of each
      std::vector<double> a(n[m], 1.0);
      if (s > 0.0 && !plan->wrap[m]) {
        const int o0 = m == 0 ? 1 : 0, o1 = m == 2 ? 1 : 2;
        const int c0 = std::min(n[o0], 24), c1 = D == 3 ? std::min(n[o1], 24) : 1;
        double mean = 0.0;
        for (int i = 0; i < n[m]; ++i) {
          double l = 0.0;
          for (int u = 0; u < c0; ++u)
            for (int v = 0; v < c1; ++v) {
              const double g0 = g[o0][(int)((2L * u + 1) * n[o0] / (2 * c0))];
              const double g1 = D == 3 ? g[o1][(int)((2L * v + 1) * n[o1] / (2 * c1))] : 0.0;
              l -= std::log(1.0 + s * (g[m][i] + g0 + g1));
            }
          a[i] = l / ((double)c0 * c1);
          mean += a[i] / n[m];
        }
        for (double& v : a) v = std::exp(v - mean);
      }
      const int other = m == 0 ? 1 : 0;
      Job job{m, q, std::vector<double>(n[m]), std::vector<double>(n[m]), false};
      for (int i = 0; i < n[m]; ++i) {
        job.kf[i] = cj[m] * f[m][m][i] * a[i];
        job.D[i] = f[other][m][i] * a[i];
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
    } catch (const std::system_error&) {
      build(b);
    }
  }
  for (std::thread& th : pool) th.join();
  for (const Job& b : jobs)
    if (!b.ok) return;
  plan->on = true;
}

}  // namespace piso
