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

// 2D layouts of unit cells: blocks as {nx, ny}, connections as {block, side, begin, end,
// other, other begin} (both directions listed), every other side Dirichlet.
struct Join { int b, side, t0, t1, o, ot0; };
static bool layout(std::vector<std::vector<int>> blocks, std::vector<Join> joins, FdmPlan* p, int* n0, int* n1) {
  std::vector<int> cells;
  std::vector<piso_side_desc> sides;
  size_t N = 0;
  for (size_t b = 0; b < blocks.size(); ++b) {
    cells.insert(cells.end(), {blocks[b][0], blocks[b][1], 1});
    N += (size_t)blocks[b][0] * blocks[b][1];
    for (int s = 0; s < 4; ++s) {
      bool any = false;
      for (const Join& j : joins) {
        if (j.b != (int)b || j.side != s) continue;
        any = true;
        piso_side_desc d{};
        d.block = j.b;
        d.side = s;
        d.kind = PISO_SIDE_CONNECT;
        d.begin[0] = j.t0;
        d.end[0] = j.t1;
        d.end[1] = 1;
        d.other_block = j.o;
        d.other_begin[0] = j.ot0;
        sides.push_back(d);
      }
      if (any) continue;
      piso_side_desc d{};
      d.block = (int)b;
      d.side = s;
      d.kind = PISO_SIDE_DIRICHLET;
      d.end[0] = blocks[b][1 - s / 2];
      d.end[1] = 1;
      sides.push_back(d);
    }
  }
  std::vector<double> T(4 * N, 0.0), J(N, 1.0);
  for (size_t P = 0; P < N; ++P) T[P] = T[3 * N + P] = 1.0;
  piso_domain_desc d{};
  d.dim = 2;
  d.n_blocks = (int)blocks.size();
  d.n_sides = (int)sides.size();
  d.block_cells = cells.data();
  d.sides = sides.data();
  d.T = T.data();
  d.J = J.data();
  Topology t;
  std::string err;
  CHECK(build_topology(&d, &t, &err) == PISO_OK, "%s", err.c_str());
  *p = FdmPlan();
  fdm_plan(&d, t, p);
  *n0 = p->n[0];
  *n1 = p->n[1];
  return p->on;
}

int main() {
  FdmPlan p;
  int n0 = 0, n1 = 0;
  // two blocks side by side; the same joined at both ends (periodic)
  CHECK(layout({{4, 3}, {6, 3}}, {{0, 1, 0, 3, 1, 0}, {1, 0, 0, 3, 0, 0}}, &p, &n0, &n1) && n0 == 10 && n1 == 3 &&
        p.cell[4] == 12 && !p.wrap[0], "two blocks");
  CHECK(layout({{4, 3}, {6, 3}}, {{0, 1, 0, 3, 1, 0}, {1, 0, 0, 3, 0, 0}, {1, 1, 0, 3, 0, 0}, {0, 0, 0, 3, 1, 0}}, &p,
               &n0, &n1) && n0 == 10 && p.wrap[0] && p.line == 1, "two blocks, periodic");
  // an annulus of 5 x 8 with four blocks of 3 x 2 around it (perm: theta becomes the first axis)
  std::vector<Join> oh = {{0, 2, 0, 5, 0, 0}, {0, 3, 0, 5, 0, 0}};
  for (int k = 0; k < 4; ++k) {
    oh.push_back({0, 1, 2 * k, 2 * k + 2, 1 + k, 0});
    oh.push_back({1 + k, 0, 0, 2, 0, 2 * k});
    oh.push_back({1 + k, 2, 0, 3, 1 + (k + 3) % 4, 0});
    oh.push_back({1 + k, 3, 0, 3, 1 + (k + 1) % 4, 0});
  }
  CHECK(layout({{5, 8}, {3, 2}, {3, 2}, {3, 2}, {3, 2}}, oh, &p, &n0, &n1) && n0 == 8 && n1 == 8 && p.wrap[0] &&
        !p.wrap[1] && p.cell[8 * 5 + 2] == 40 + 6, "annulus and transition blocks");
  // three blocks in an L
  CHECK(!layout({{4, 4}, {4, 4}, {4, 4}}, {{0, 1, 0, 4, 1, 0}, {1, 0, 0, 4, 0, 0}, {0, 3, 0, 4, 2, 0}, {2, 2, 0, 4, 0, 0}},
                &p, &n0, &n1), "L of three blocks");
  // four blocks around a point, one pair not joined (a slit inside the box)
  CHECK(!layout({{4, 4}, {4, 4}, {4, 4}, {4, 4}},
                {{0, 1, 0, 4, 1, 0}, {1, 0, 0, 4, 0, 0}, {0, 3, 0, 4, 2, 0}, {2, 2, 0, 4, 0, 0}, {1, 3, 0, 4, 3, 0},
                 {3, 2, 0, 4, 1, 0}}, &p, &n0, &n1), "slit");
  p = FdmPlan();
  CHECK(plan_of({uniform(12, .5), stretched(17), uniform(9, .3)}, 5, 1.0, &p) && p.rungs == 1 && p.line == 1, "channel");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({stretched(70), stretched(33)}, 0, 1.0, &p) && p.rungs == kFdmRungs && p.line == 1, "cavity");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({stretched(9), uniform(8, .5), stretched(33)}, 2, 1.0, &p) && p.line == 2, "lines along z");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({stretched(33), uniform(8, .5)}, 2, 1.0, &p) && p.line == 1 && p.perm[0] == 1 && !p.plain &&
        p.n[0] == 8 && p.cell[1] == 33, "x and y exchanged");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({uniform(6, .5), uniform(1, .5), uniform(2, 1.0)}, 7, 1.0, &p) && p.rungs == 1 && p.line == -1, "box");
  diagonal(p);
  p = FdmPlan();
  CHECK(plan_of({uniform(kFdmMaxN, .5), uniform(2, .5)}, 1, 1.0, &p), "longest axis");
  p = FdmPlan();
  CHECK(!plan_of({uniform(kFdmMaxN + 1, .5), uniform(2, .5)}, 1, 1.0, &p), "too long");
  p = FdmPlan();
  CHECK(plan_of({uniform(8, .5), stretched(8)}, 1, 1.5, &p), "nearly a product");
  p = FdmPlan();
  CHECK(!plan_of({uniform(8, .5), stretched(8)}, 1, 400.0, &p), "no product");
  std::printf("%s (%d failures)\n", failures ? "FAILED" : "passed", failures);
  return failures != 0;
}
