// Solver of the global coarse operator E_0 (gcoarse.hpp) by nested dissection.
//
// E_0 is real and couples a coarse node to its 3 x 3 neighbours.  It is solved exactly in FP64 by nested
// dissection: a box of the coarse grid is split by a cross of grid lines (the separator) into four
// boxes, down to boxes of at most 10 x 10 nodes.  With S the separator of a box (all of its nodes
// for a smallest one) and R the ring of nodes around the box, which belong to the separators of
// larger boxes, the elimination of everything inside the box leaves a dense front on S and R:
//   F = E_0's entries in rows or columns of S + the children's update matrices,
//   Binv = F_SS^{-1},  W = F_RS Binv,  update matrix U = F_RR - W F_SR.
// The solve is then, one launch per depth and direction,
//   from the smallest boxes up:  y_S = b_S + sum of the children's g,  g_R = (children's g) - W y_S;
//   from the largest box down:   x_S = Binv y_S - W^T x_R.
// Every launch is a batch of independent dense products spread over the whole chip, and their
// number is 2 log2(n / 10) + 1 for n x n unknowns (11 at n = 317).  The two matrices kept of a box of width w
// that is cut inside the grid (s = 2 w, b = 4 w) hold s b + s (s + b) = 20 w^2 values, whatever its depth (12 w^2 for the
// four below the whole grid, 4 w^2 for that), so the factors grow as n^2 log n; a smallest box holds about 166 w^2,
// 103 of the 156 MB at n = 317.
// (The block cyclic reduction over the grid's rows has n^3: at n = 317 it reads 0.90 GB per solve in
// 21 launches.)
// The set-up inverts F_SS by block Gauss-Jordan sweeps, batched over the boxes of a depth, with partial
// pivoting inside each pivot block of at most 56 unknowns.  Between the blocks there is no
// pivoting, and a part of a separator can be nearly singular (n = 317, k = 200: entries of 460
// in a pivot inverse, 1e-9 off the identity), so one Newton step X <- X + X (I - F_SS X)
// follows, which squares that error; it leaves a smaller one than an inverse with pivoting over the
// whole separator (3e-13 against 2e-12 of the solution on that grid).
// Between boxes there is no pivoting either (nor was there in the cyclic reduction), and k^2 near an
// eigenvalue of some box costs digits.  The set-up therefore solves for a pseudo-random vector,
// refines the solution once and takes the correction for the error.  A handle where that exceeds
// kNdRefineAbove refines every solve: r = b - E_0 x, x <- x + E_0^{-1} r, which squares it; above
// kNdRefuseAbove that would not be enough and the caller takes the cyclic reduction, whose pivots
// are other matrices.  Relative errors of the solve over eleven grids from n = 15 to 636: cyclic
// reduction 2e-14 to 4e-8, this without refinement 3e-15 to 4e-10, with the rule at most 3e-12.
#pragma once

#include <vector>

#include "common.hpp"

namespace ddh {

constexpr int kNdRhsGroup = 4;          // right-hand sides per pass of the solve kernel
constexpr int kNdLeaf = 10;             // largest box that is eliminated as a whole
constexpr int kNdPivot = 56;            // largest pivot block of the set-up's elimination (LDS: 64 KB)
constexpr int kNdTile = 64;             // rows and columns of a front per workgroup of the set-up
constexpr int kNdChildren = 4;
constexpr double kNdRefineAbove = 3e-12;
constexpr double kNdRefuseAbove = 1e-6;

// One box: s separator nodes, then b ring nodes (positions 0 .. m-1 of its front, m = s + b).
struct NdNode {
  int s, b;
  int idx;                  // offset of its node list (grid indices) and of its child positions
  int g;                    // offset of its ring values g in the update vectors
  int kids;                 // children, their node numbers consecutive from `kid`
  int kid;
  long long up, down;       // offsets of the solve matrices: [-W] (b x s), [Binv | -W^T] (s x m), both
                            // stored column by column
  long long front;          // offset of the front in its depth's set-up buffer (m x m, row-major)
  long long inv;            // offset of its separator's matrices in the set-up buffers (s x s, row-major)
  int panel;                // offset of its panels in the set-up buffers (rows)
  int steps;                // pivot blocks
};

struct NdLevel {
  int first, count;         // nodes [first, first + count)
  int max_s, max_b, steps;
};

// Device memory freed with the object.  Small requests share an allocation, large ones have their own: set-up of a
// handle with a 9 x 9 coarse grid 783 us with one each and 755 shared, with a 39 x 39 one 1.8 ms
// and 2.3 with everything in one.
constexpr size_t kNdSmall = 128 << 10, kNdChunk = 512 << 10;

class NdMemory {
 public:
  NdMemory() = default;
  NdMemory(const NdMemory&) = delete;
  NdMemory& operator=(const NdMemory&) = delete;
  ~NdMemory();
  template <typename T>
  hipError_t take(T** p, size_t count) {
    return take((void**)p, count * sizeof(T));
  }

 private:
  hipError_t take(void** p, size_t bytes);
  std::vector<void*> blocks;
  unsigned char* chunk = nullptr;
  size_t room = 0;
};

class NestedDissection {
 public:
  double min_pivot = 0.0;
  bool accurate = false;         // finite, and solve_error at most kNdRefuseAbove
  bool refine = false;           // refine every solve once
  double solve_error = 0.0;      // estimated at set-up, before refinement
  long long solve_bytes = 0;     // algorithmic traffic of one solve

  // Factor the n x n grid's operator E ([n n][9], kept by the caller) for solves on the vectors cv
  // ([nr][2 n n], b | x); synchronises st.  Not to be used if it leaves `accurate` false.
  hipError_t setup(const double* E, int n, int nr, cplx<double>* cv, hipStream_t st);
  // x = E_0^{-1} b for the first nr right-hand sides.
  hipError_t solve(int nr, hipStream_t st);

 private:
  int nc = 0;
  long long ncoarse = 0, nfac = 0, glen = 0, nidx = 0;
  const double* E0c = nullptr;
  cplx<double>* cv = nullptr;
  // device
  double* fac = nullptr;         // factors (real: A and Z_0 are real)
  NdNode* nodes = nullptr;
  int* idx = nullptr;            // grid indices of every front
  int* cpos = nullptr;           // [kNdChildren][...] where a front position receives a child's g, or -1
  cplx<double>* yv = nullptr;    // [nrhs][ncoarse] y of the upward pass
  cplx<double>* gv = nullptr;    // [nrhs][glen] update vectors
  cplx<double>* rv = nullptr;    // [nrhs][2 ncoarse] residual | correction
  std::vector<NdLevel> levels;   // by depth, the whole grid first
  NdMemory memory;               // holds the arrays above

  hipError_t residual(int nr, hipStream_t st);   // rv = b - E_0 x
  hipError_t sweep(const cplx<double>* b, long long bstride, cplx<double>* x, long long xstride, int nr, hipStream_t st);
};

}  // namespace ddh
