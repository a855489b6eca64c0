// Host check of the fast-diagonalisation plan: the 1D bases diagonalise the operators whose
// weights the plan states, and grids that are no tensor-product block are turned down.
// Built and run by tests/test_fdm_plan.py under AddressSanitizer and UBSan.
#include <cmath>
#include <cstdio>
#include <vector>

#include "../../paper_2505_16992_amd/csrc/piso_fdm_plan.h"

using namespace piso;

static int failures = 0;
#define CHECK(c, ...) \
  do { if (!(c)) { ++failures; std::printf("FAIL %s: ", #c); std::printf(__VA_ARGS__); std::printf("\n"); } } while (0)

// One block from 1D cell widths; wrap bit m: axis m periodic.  bend scales one cell's J.
static bool plan_of(std::vector<std::vector<double>> w, int wrap, double bend, FdmPlan* p) {
  const int D = (int)w.size();
  if (D == 2) w.push_back({1.0});
  const int n[3] = {(int)w[0].size(), (int)w[1].size(), (int)w[2].size()};
  const size_t N = (size_t)n[0] * n[1] * n[2];
  std::vector<double> T(D * D * N, 0.0), J(N, 1.0);
  for (size_t P = 0; P < N; ++P) {
    const int i[3] = {(int)(P % n[0]), (int)(P / n[0] % n[1]), (int)(P / n[0] / n[1])};
    for (int m = 0; m < D; ++m) {
      T[(size_t)(m * D + m) * N + P] = 1.0 / w[m][i[m]];
      J[P] *= w[m][i[m]];
    }
  }
  J[N / 2] *= bend;
  std::vector<piso_side_desc> sides;
  for (int s = 0; s < 2 * D; ++s) {
    piso_side_desc d{};
    d.side = s;
    d.kind = (wrap >> (s / 2)) & 1 ? PISO_SIDE_CONNECT : PISO_SIDE_DIRICHLET;
    int e[2] = {1, 1}, q = 0;
    for (int a = 0; a < D; ++a)
      if (a != s / 2) e[q++] = n[a];
    d.end[0] = e[0];
    d.end[1] = e[1];
    sides.push_back(d);
  }
  piso_domain_desc d{};
  d.dim = D;
  d.n_blocks = 1;
  d.n_sides = (int)sides.size();
  d.block_cells = n;
  d.sides = sides.data();
  d.T = T.data();
  d.J = J.data();
  Topology t;
  std::string err;
  CHECK(build_topology(&d, &t, &err) == PISO_OK, "%s", err.c_str());
  fdm_plan(&d, t, p);
  return p->on;
}

// V^T D V = I and V^T K V = diag(lam) with the weights of the plan.
static void diagonal(const FdmPlan& p) {
  for (int m = 0; m < p.dim; ++m)
    for (int q = 0; m != p.line && q < p.rungs; ++q) {
      const int n = p.n[m], o = m == 0 ? 1 : 0;
      const double *D = &p.wt[o][m][(size_t)q * n], *K = &p.wt[m][m][(size_t)q * n];
      const double* V = &p.V[m][(size_t)q * n * n];
      const double* lam = &p.lam[m][(size_t)q * n];
      double worst = 0.0, top = 1e-300;
      for (int k = 0; k < n; ++k) top = std::fmax(top, lam[k]);
      for (int k = 0; k < n; ++k)
        for (int l = 0; l < n; ++l) {
          double d = 0.0, s = 0.0;
          for (int i = 0; i < n; ++i) {
            d += V[i * n + k] * D[i] * V[i * n + l];
            const int r = i + 1 < n ? i + 1 : 0;
            if (i + 1 < n || p.wrap[m]) s += K[i] * (V[i * n + k] - V[r * n + k]) * (V[i * n + l] - V[r * n + l]);
          }
          worst = std::fmax(worst, std::fabs(d - (k == l)));
          worst = std::fmax(worst, std::fabs(s - (k == l ? lam[k] : 0.0)) / top);
        }
      CHECK(worst < 1e-11 && lam[0] == 0.0, "axis %d rung %d n %d: %.2e", m, q, n, worst);
    }
}

static std::vector<double> uniform(int n, double h) { return std::vector<double>(n, h); }
static std::vector<double> stretched(int n) {
  std::vector<double> w(n);
  for (int i = 0; i < n; ++i) w[i] = std::tanh(1.5 * (2.0 * (i + 1) / n - 1)) - std::tanh(1.5 * (2.0 * i / n - 1));
  return w;
}

int main() {
  FdmPlan p;
  CHECK(plan_of({uniform(12, .5), stretched(17), uniform(9, .3)}, 5, 1.0, &p) && p.rungs == 1 && p.line == 1, "channel");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({stretched(70), stretched(33)}, 0, 1.0, &p) && p.rungs == kFdmRungs && p.line == 1, "cavity");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({stretched(9), uniform(8, .5), stretched(33)}, 2, 1.0, &p) && p.line == 2, "lines along z");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({stretched(33), uniform(8, .5)}, 2, 1.0, &p) && p.line == -1 && p.rungs == kFdmRungs, "no line axis");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({uniform(6, .5), uniform(1, .5), uniform(2, 1.0)}, 7, 1.0, &p) && p.rungs == 1 && p.line == -1, "box");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({uniform(kFdmMaxN, .5), uniform(2, .5)}, 1, 1.0, &p), "longest axis");
  p = FdmPlan();
  CHECK(!plan_of({uniform(kFdmMaxN + 1, .5), uniform(2, .5)}, 1, 1.0, &p), "too long");
  p = FdmPlan();
  CHECK(!plan_of({stretched(8), uniform(8, .5)}, 3, 1.0, &p), "stretched periodic axis");
  p = FdmPlan();
  CHECK(!plan_of({uniform(8, .5), stretched(8)}, 1, 1.001, &p), "no tensor product");
  std::printf("%s (%d failures)\n", failures ? "FAILED" : "passed", failures);
  return failures != 0;
}
