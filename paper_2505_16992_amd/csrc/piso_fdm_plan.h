// Fast-diagonalisation plan of a logical box (host side of piso_fdm.hip): 1D generalised
// eigenbases in which the pressure operator of a tensor-product grid is diagonal.  Plain
// C++ without HIP.
//
// The box.  Connections keep the axes' orientation, so many multi-block layouts are one
// logical box cut into blocks: a block's position follows from its neighbours'.  The annulus
// of a cylinder O-H grid and its four transition blocks are a box of n_r + n_out by n_theta
// cells, periodic in theta.  `cell` maps the box to the cells.
//
// M = -P has the face weights lerp(alpha_jj / A).  Where alpha_jj(i0, i1, i2) is a product of
// one factor per axis (or replaced by one: means of the logarithm) and 1 / A is replaced by
// a product a_0(i0) a_1(i1) a_2(i2),
//   M0 = sum_j K_j (x) (x)_{m != j} D_m,    K_m: 1D stiffness, D_m: 1D weights,
// and with K_m V_m = D_m V_m diag(lambda_m), V_m^T D_m V_m = I (columns of V_m),
//   M0^+ = ((x) V_m) diag(1 / sum_m lambda_m) ((x) V_m)^T   (null mode left out):
// one small dense product per axis and direction, exact for M0.  The scale of M0 does not
// matter to the conjugate gradients, only its shape.
//
// One axis with walls, the line axis, needs no basis: there the transformed system is one
// tridiagonal system per mode of the other axes, whose coefficients (one profile per term)
// are the plane means of the operator's own face weights.  1 / A then may vary along that
// axis in any way.  (A channel's 1 / A varies with the wall distance alone: a 32 x 24 x 16
// one converges by 5e-6 per iteration with its profile and by 8e-4 with a constant.)
//
// Along the other axes 1 / A varies with the grid (A = 1/dt + nu g, g from the metrics) as
// far as nu dt g is comparable to one and the axis has walls, so a plan holds a ladder of
// bases for fixed values of nu dt max(g); the operator's face weights choose the rung on
// the device.
#pragma once

#include <cstdint>
#include <vector>

#include "../../include/piso.h"
#include "piso_topology.h"

namespace piso {

constexpr int kFdmRungs = 6;
// nu dt max(g) of the rungs.  256^2 cavity at 17: spread of the face-weight ratios 16.5 with
// the first rung, 2.3 with 8, 3.6 with 34; 49 x 17 open channel at 1.2: 2.15 and 1.16.
constexpr double kFdmLadder[kFdmRungs] = {0.0, 0.1, 0.4, 1.5, 8.0, 50.0};
constexpr int kFdmMaxN = 512;   // longest axis: dense bases cost n^2, their construction n^3
// Largest spread of the metric alone (1 / A constant) that gets a plan: the cylinder's O-H
// grid has 2.2 (10 iterations to 1e-7 where the V-cycle takes 46), tensor products 1.
constexpr double kFdmMaxShape = 8.0;

struct FdmPlan {
  bool on = false;
  int dim = 0, rungs = 1;          // rungs: 1 where the metrics give 1 / A no shape
  // axis m of the box is axis perm[m] of the blocks: the line axis is never the box's first
  int perm[3] = {0, 1, 2};
  std::vector<int> cell;           // cell of each box position, first axis fastest
  bool plain = true;               // cell is the identity
  int n[3] = {1, 1, 1};
  bool wrap[3] = {false, false, false};
  int line = -1;                   // axis of the tridiagonal systems (1 or 2), -1: none
  // per axis m != line and rung q, at [q * n + i] (V: [(q * n + i) * n + k])
  std::vector<double> lam[3];      // lambda_m[k], ascending, lam[0] = 0 exactly
  std::vector<double> V[3];
  // 1D factors of M0's face weights (ones along the line axis): weight of the face above
  // cell (i0, i1, i2) along j = prod_m wt[j][m][q * n_m + i_m], times the profile of term j
  std::vector<double> wt[3][3];
};

// Leaves plan->on false where the blocks are no box whose sides are walls or wrap onto the
// box, an axis is too long, or the metric is too far from a product.  Throws only
// std::bad_alloc.
void fdm_plan(const piso_domain_desc* d, const Topology& topo, FdmPlan* plan);

// Eigenvalues (ascending) and orthonormal eigenvectors of the symmetric tridiagonal matrix
// with diagonal a[n] and off-diagonal b[n - 1]: z[i * n + k] is component i of vector k.
// False if an eigenvalue does not settle.
bool tridiag_eigen(std::vector<double> a, std::vector<double> b, std::vector<double>* w, std::vector<double>* z);

}  // namespace piso
