// Host memory running out while the fast-diagonalisation plan is built: every allocation in turn
// fails, also those that start a thread.  fdm_plan throws std::bad_alloc or leaves no plan; it
// must not end the process (a joinable thread that goes out of scope does).  Built and run by
// tests/test_fdm_plan_memory.py.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "../../paper_2505_16992_amd/csrc/piso_fdm_plan.h"

static std::atomic<long> g_left{-1};   // allocations until one fails (negative: none does)
static std::atomic<bool> g_failed{false};

void* operator new(std::size_t n) {
  if (g_left.load() >= 0 && g_left.fetch_sub(1) == 0) {
    g_failed = true;
    throw std::bad_alloc();
  }
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
  // walls all around, cells enough for the threads of the metric's scan, axes long enough for
  // those of the bases
  const int nx = 200, ny = 512, N = nx * ny;
  std::vector<double> T(4 * (size_t)N, 0.0), J(N, 1.0);
  for (int P = 0; P < N; ++P) T[P] = T[3 * (size_t)N + P] = 1.0 + 0.5 * (P % nx) / nx;
  const int cells[3] = {nx, ny, 1};
  std::vector<piso_side_desc> sides(4);
  for (int s = 0; s < 4; ++s) {
    sides[s] = piso_side_desc{};
    sides[s].side = s;
    sides[s].kind = PISO_SIDE_DIRICHLET;
    sides[s].end[0] = s < 2 ? ny : nx;
    sides[s].end[1] = 1;
  }
  piso_domain_desc d{};
  d.dim = 2;
  d.n_blocks = 1;
  d.n_sides = 4;
  d.block_cells = cells;
  d.sides = sides.data();
  d.T = T.data();
  d.J = J.data();
  piso::Topology t;
  std::string err;
  if (piso::build_topology(&d, &t, &err) != PISO_OK) return 2;
  int thrown = 0, none = 0, runs = 0;
  for (long k = 0;; ++k, ++runs) {
    piso::FdmPlan p;
    g_failed = false;
    g_left = k;
    try {
      piso::fdm_plan(&d, t, &p);
    } catch (const std::bad_alloc&) {
      ++thrown;
    }
    g_left = -1;
    if (!g_failed) {   // fewer allocations than k: the plan is there
      if (!p.on) return 3;
      break;
    }
    if (!p.on) ++none;
  }
  std::printf("%d failing allocations: %d thrown, %d without a plan\n", runs, thrown, none);
  return runs > 20 && thrown > 0 ? 0 : 4;
}
