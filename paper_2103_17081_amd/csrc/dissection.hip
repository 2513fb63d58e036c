// Nested dissection of the global coarse operator: plan, set-up kernels and solve (definitions in
// dissection.hpp).
#include "dissection.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

#include "outer.hpp"

namespace ddh {

namespace {

// ---- set-up: fronts --------------------------------------------------------------------

// Fronts of one depth: F(i, j) = E_0 entry if i or j is a separator node, plus the children's
// update matrices where both positions receive them; X starts as a copy of F_SS.
__global__ void __launch_bounds__(256) nd_front_kernel(const NdNode* __restrict__ nodes, int first,
                                                       const int* __restrict__ idx, const int* __restrict__ cpos,
                                                       long long nidx, const double* __restrict__ E0c, int n,
                                                       const double* __restrict__ kids, double* __restrict__ fronts,
                                                       double* __restrict__ X) {
  const NdNode nd = nodes[first + blockIdx.y];
  const int m = nd.s + nd.b;
  const long long mm = (long long)m * m;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < mm; e += gridDim.x * 256ll) {
    const int i = (int)(e / m), j = (int)(e - (long long)i * m);
    double v = 0.0;
    if (i < nd.s || j < nd.s) {
      const int gi = idx[nd.idx + i], gj = idx[nd.idx + j];
      const int dx = gj % n - gi % n, dy = gj / n - gi / n;
      if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1) v = E0c[(long long)gi * 9 + 3 * (dy + 1) + (dx + 1)];
    }
    for (int c = 0; c < nd.kids; ++c) {
      const int pi = cpos[c * nidx + nd.idx + i], pj = cpos[c * nidx + nd.idx + j];
      if (pi >= 0 && pj >= 0) {
        const NdNode kd = nodes[nd.kid + c];
        const int km = kd.s + kd.b;
        v += kids[kd.front + (long long)(kd.s + pi - kd.g) * km + (kd.s + pj - kd.g)];
      }
    }
    fronts[nd.front + e] = v;
    if (i < nd.s && j < nd.s) X[nd.inv + (long long)i * nd.s + j] = v;
  }
}

// Pivot block of elimination step t: unknowns [p0, p0 + pn) of the separator (pn = 0: none left).
__device__ __forceinline__ void nd_pivot(const NdNode& nd, int t, int& p0, int& pn) {
  const int w = (nd.s + nd.steps - 1) / nd.steps;
  p0 = min(t * w, nd.s);
  pn = min(w, nd.s - p0);
}

// Largest v of the wave in every lane (no NaN).
__device__ __forceinline__ double nd_wave_max(double v) {
  v = fmax(v, dpp_f64<kDppXor1>(v));
  v = fmax(v, dpp_f64<kDppXor2>(v));
  v = fmax(v, dpp_f64<kDppHalfMirror>(v));
  v = fmax(v, dpp_f64<kDppMirror>(v));
  const auto larger = [](auto lo, auto hi) { return fmax(join_f64(lo[0], hi[0]), join_f64(lo[1], hi[1])); };
  unsigned long long x = (unsigned long long)__double_as_longlong(v);
  unsigned lo = (unsigned)x, hi = (unsigned)(x >> 32);
  v = larger(__builtin_amdgcn_permlane16_swap(lo, lo, false, false), __builtin_amdgcn_permlane16_swap(hi, hi, false, false));
  x = (unsigned long long)__double_as_longlong(v);
  lo = (unsigned)x;
  hi = (unsigned)(x >> 32);
  return larger(__builtin_amdgcn_permlane32_swap(lo, lo, false, false), __builtin_amdgcn_permlane32_swap(hi, hi, false, false));
}

// Inverse of each separator matrix's pivot block in LDS: Gauss-Jordan with partial pivoting, one
// workgroup per box; piv[node] keeps the smallest |pivot| (NaN sticks).  A serial chain of n steps: every wave
// finds the pivot for itself, reads what it needs of the two rows and the column, and writes its entries, interchange included,
// after one barrier.  Set-up of a handle with a 10 x 10 coarse grid (two blocks of 50): 960 us with five barriers a step,
// now 863.
__global__ void __launch_bounds__(256) nd_pivot_kernel(const NdNode* __restrict__ nodes, int first, int t,
                                                       const double* __restrict__ X, double* __restrict__ dinv,
                                                       double* __restrict__ piv) {
  const NdNode nd = nodes[first + blockIdx.x];
  int p0, n;
  nd_pivot(nd, t, p0, n);
  if (n <= 0) return;
  __shared__ double A[kNdPivot][kNdPivot + 1];
  constexpr int kRows = kNdPivot / 4;
  const int tid = threadIdx.x, m = nd.s, c = tid % kWave, r0 = tid / kWave, cc = min(c, n - 1);
  const double* F = X + nd.inv + (long long)p0 * m + p0;
  for (int r = r0; r < n; r += 4)
    if (c < n) A[r][c] = F[(long long)r * m + c];
  double minp = INFINITY;
  int perm = 0;   // lane p: the row that step p took
  __syncthreads();
  for (int p = 0; p < n; ++p) {
    const double v = fabs(A[cc][p]), cand = c >= p && c < n && v == v ? v : -1.0;
    const double best = nd_wave_max(cand);
    const unsigned long long at = __ballot(cand == best);
    const bool valid = best >= 0.0;   // (not in a column of NaN)
    const int q = valid ? __builtin_ctzll(at) : p;
    const double pmax = valid ? best : NAN;
    minp = pmax < minp || pmax != pmax ? pmax : minp;
    if (c == p) perm = q;
    // entries of rows p and q in this lane's column, and of column p in this wave's rows
    const double top = A[p][cc], inv = 1.0 / A[q][p], row = cc == p ? inv : inv * A[q][cc], topp = A[p][p];
    double own[kRows], col[kRows];
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const int r = min(r0 + 4 * i, n - 1);
      own[i] = r == q ? top : A[r][cc];
      col[i] = r == q ? topp : A[r][p];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const int r = r0 + 4 * i;
      if (r < n && c < n) A[r][c] = r == p ? row : (c == p ? -inv * col[i] : own[i] - row * col[i]);
    }
    __syncthreads();
  }
  // undo the row interchanges: columns swapped in reverse order
  int src = c;
  for (int p = n - 1; p >= 0; --p) {
    const int q = __builtin_amdgcn_readlane(perm, p);
    const int sp = __builtin_amdgcn_readlane(src, p), sq = __builtin_amdgcn_readlane(src, q);
    src = c == p ? sq : (c == q ? sp : src);
  }
  double* D = dinv + (long long)blockIdx.x * kNdPivot * kNdPivot;
  for (int r = r0; r < n; r += 4)
    if (c < n) D[r * kNdPivot + c] = A[r][src];
  if (tid == 0) {
    const double o = t > 0 ? piv[first + blockIdx.x] : INFINITY;
    piv[first + blockIdx.x] = minp < o || minp != minp ? minp : o;
  }
}

// Panels of an elimination step: rows = Dinv X_p: (Dinv itself in the pivot columns), cols = X_:p,
// 64 columns and rows of the matrix per workgroup.
__global__ void __launch_bounds__(256) nd_panel_kernel(const NdNode* __restrict__ nodes, int first, int t,
                                                       const double* __restrict__ X,
                                                       const double* __restrict__ dinv, double* __restrict__ rows,
                                                       double* __restrict__ cols) {
  const NdNode nd = nodes[first + blockIdx.y];
  int p0, pn;
  nd_pivot(nd, t, p0, pn);
  const int m = nd.s, j0 = blockIdx.x * kNdTile;
  if (pn <= 0 || j0 >= m) return;
  __shared__ double D[kNdPivot][kNdPivot], P[kNdPivot][kNdTile];
  const int tid = threadIdx.x, c = tid % kNdTile, r0 = tid / kNdTile, j = j0 + c;
  const double* F = X + nd.inv;
  const double* Di = dinv + (long long)blockIdx.y * kNdPivot * kNdPivot;
  double* Rp = rows + (long long)nd.panel * kNdPivot;   // pivot row k at k m
  double* Cp = cols + (long long)nd.panel * kNdPivot;   // row i at i kNdPivot
  for (int k = r0; k < pn; k += 4) {
    if (c < pn) D[k][c] = Di[k * kNdPivot + c];
    P[k][c] = j < m ? F[(long long)(p0 + k) * m + j] : 0.0;
  }
  for (int i = r0; i < kNdTile && j0 + i < m; i += 4)
    if (c < pn) Cp[(long long)(j0 + i) * kNdPivot + c] = F[(long long)(j0 + i) * m + p0 + c];
  __syncthreads();
  if (j >= m) return;
  for (int k = r0; k < pn; k += 4) {
    double v = 0.0;
    if (j >= p0 && j < p0 + pn) {
      v = D[k][j - p0];
    } else {
      for (int l = 0; l < pn; ++l) v = fma(D[k][l], P[l][c], v);
    }
    Rp[(long long)k * m + j] = v;
  }
}

// The step itself, 64 x 64 entries of the matrix per workgroup, 4 x 4 per thread:
// X_ij -= cols_i rows_j, X_ip = -cols_i Dinv, X_p: = rows.
__global__ void __launch_bounds__(256) nd_eliminate_kernel(const NdNode* __restrict__ nodes, int first, int t,
                                                           double* __restrict__ X,
                                                           const double* __restrict__ rows,
                                                           const double* __restrict__ cols) {
  const NdNode nd = nodes[first + blockIdx.y];
  int p0, pn;
  nd_pivot(nd, t, p0, pn);
  const int m = nd.s, tiles = (m + kNdTile - 1) / kNdTile;
  if (pn <= 0 || (int)blockIdx.x >= tiles * tiles) return;
  const int i0 = (blockIdx.x / tiles) * kNdTile, j0 = (blockIdx.x % tiles) * kNdTile;
  __shared__ double Cs[kNdTile][kNdPivot + 1], Rs[kNdPivot][kNdTile];
  const int tid = threadIdx.x, lx = tid % kNdTile, ly = tid / kNdTile;
  const double* Rp = rows + (long long)nd.panel * kNdPivot;
  const double* Cp = cols + (long long)nd.panel * kNdPivot;
  for (int q = ly; q < kNdTile; q += 4) {
    if (lx < pn) Cs[q][lx] = i0 + q < m ? Cp[(long long)(i0 + q) * kNdPivot + lx] : 0.0;
    if (q < pn) Rs[q][lx] = j0 + lx < m ? Rp[(long long)q * m + j0 + lx] : 0.0;
  }
  __syncthreads();
  const int ty = tid / 16, tx = tid % 16;
  double acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
  for (int k = 0; k < pn; ++k) {
    double a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = Cs[ty + 16 * i][k];
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = Rs[k][tx + 16 * j];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = fma(a[i], b[j], acc[i][j]);
  }
  double* F = X + nd.inv;
#pragma unroll
  for (int ii = 0; ii < 4; ++ii) {
    const int i = i0 + ty + 16 * ii;
    if (i >= m) continue;
    const bool ip = i >= p0 && i < p0 + pn;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int j = j0 + tx + 16 * jj;
      if (j >= m) continue;
      const bool jp = j >= p0 && j < p0 + pn;
      const long long e = (long long)i * m + j;
      F[e] = ip ? Rp[(long long)(i - p0) * m + j] : (jp ? -acc[ii][jj] : F[e] - acc[ii][jj]);
    }
  }
}

// Products of a depth's boxes, 64 x 64 entries per workgroup, 4 x 4 per thread, 16 of the inner
// dimension at a time through LDS:
//   mode 0: T = I - F_SS X;  1: Y = X + X T;  2: up = -Y F_SR (row-major s x b: (-W)^T);
//   3: F_RR += F_RS up (the update matrix U).
constexpr int kGK = 16;
__global__ void __launch_bounds__(256) nd_product_kernel(const NdNode* __restrict__ nodes, int first, int mode,
                                                         double* fronts, const double* X, double* T, double* Y,
                                                         double* fac) {
  const NdNode nd = nodes[first + blockIdx.y];
  const int s = nd.s, b = nd.b, m = s + b;
  double* F = fronts + nd.front;
  const double *A, *B;
  double* C;
  int R, N, lda, ldb, ldc;
  const int K = s;
  if (mode == 0) { A = F; lda = m; B = X + nd.inv; ldb = s; C = T + nd.inv; ldc = s; R = s; N = s; }
  else if (mode == 1) { A = X + nd.inv; lda = s; B = T + nd.inv; ldb = s; C = Y + nd.inv; ldc = s; R = s; N = s; }
  else if (mode == 2) { A = Y + nd.inv; lda = s; B = F + s; ldb = m; C = fac + nd.up; ldc = b; R = s; N = b; }
  else { A = F + (long long)s * m; lda = m; B = fac + nd.up; ldb = b; C = F + (long long)s * m + s; ldc = m; R = b; N = b; }
  const int tiles = (N + kNdTile - 1) / kNdTile;
  const int r0 = (int)(blockIdx.x / max(tiles, 1)) * kNdTile, c0 = (int)(blockIdx.x % max(tiles, 1)) * kNdTile;
  if (r0 >= R || c0 >= N) return;
  __shared__ double As[kGK][kNdTile + 1];
  __shared__ double Bs[kGK][kNdTile];
  const int tid = threadIdx.x, ty = tid / 16, tx = tid % 16;
  double acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
  for (int k0 = 0; k0 < K; k0 += kGK) {
    for (int e = tid; e < kNdTile * kGK; e += 256) {
      const int r = e / kGK, k = e % kGK;
      As[k][r] = (r0 + r < R && k0 + k < K) ? A[(long long)(r0 + r) * lda + k0 + k] : 0.0;
    }
    for (int e = tid; e < kGK * kNdTile; e += 256) {
      const int k = e / kNdTile, c = e % kNdTile;
      Bs[k][c] = (k0 + k < K && c0 + c < N) ? B[(long long)(k0 + k) * ldb + c0 + c] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kGK; ++k) {
      double av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = As[k][ty + 16 * i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bv[j] = Bs[k][tx + 16 * j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fma(av[i], bv[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + ty + 16 * i;
    if (r >= R) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = c0 + tx + 16 * j;
      if (c >= N) continue;
      double* o = C + (long long)r * ldc + c;
      if (mode == 0) *o = (r == c ? 1.0 : 0.0) - acc[i][j];
      else if (mode == 1) *o = A[(long long)r * lda + c] + acc[i][j];
      else if (mode == 2) *o = -acc[i][j];
      else *o += acc[i][j];
    }
  }
}

// down(k, j) at j s + k: Binv, then -W^T (`up` transposed; F and Binv are symmetric).
__global__ void __launch_bounds__(256) nd_extract_kernel(const NdNode* __restrict__ nodes, int first,
                                                         const double* __restrict__ Y, double* __restrict__ fac) {
  const NdNode nd = nodes[first + blockIdx.y];
  const int s = nd.s, b = nd.b, m = s + b;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < (long long)s * m; e += gridDim.x * 256ll) {
    const int j = (int)(e / s), k = (int)(e - (long long)j * s);
    fac[nd.down + e] = j < s ? Y[nd.inv + (long long)k * s + j] : fac[nd.up + (long long)k * b + (j - s)];
  }
}

// ---- solve -------------------------------------------------------------------------------

struct NdVectors {
  const cplx<double>* b;
  long long bstride;
  cplx<double>* x;
  long long xstride;
  cplx<double>* y;
  long long ystride;
  cplx<double>* g;
  long long gstride;
};

// Value of front position f before this box's own product: b there (separator nodes only) plus
// what the children pass up.
__device__ __forceinline__ cplx<double> nd_received(const NdNode& nd, const int* __restrict__ idx,
                                                    const int* __restrict__ cpos, long long nidx, const NdVectors& v,
                                                    int rhs, int f) {
  cplx<double> r = czero<double>();
  if (f < nd.s) r = v.b[rhs * v.bstride + idx[nd.idx + f]];
  int p[kNdChildren];
#pragma unroll
  for (int c = 0; c < kNdChildren; ++c) p[c] = c < nd.kids ? cpos[c * nidx + nd.idx + f] : -1;
#pragma unroll
  for (int c = 0; c < kNdChildren; ++c)
    if (p[c] >= 0) r = r + v.g[rhs * v.gstride + p[c]];
  return r;
}

// One depth of the solve in one direction: box blockIdx.y, output rows [blockIdx.x Rows, + Rows).
// The input vector of a group of right-hand sides is gathered into LDS; lane r of each of the 256 / Rows
// column slices owns an output row and reads its matrix column by column (coalesced over r), the
// first Cols columns issued before the gather; the slices are summed through LDS.
// Bound by latency at most depths (dependent gathers, one launch per depth: 8 - 10 us), by the factor
// bytes at the deepest ones.  One solve, us, block cyclic reduction -> this: n = 79 75 -> 41, n = 317
// 338 -> 109 (156 MB), n = 636 1814 -> 294 (693 MB; 610 refined); set-up of a handle, ms: n = 317 139 -> 41, n = 636
// (four right-hand sides) 1353 -> 33.
template <int Rows, int Cols>
__global__ void __launch_bounds__(256) nd_solve_kernel(const NdNode* __restrict__ nodes, int first,
                                                       const int* __restrict__ idx, const int* __restrict__ cpos,
                                                       long long nidx, const double* __restrict__ fac, NdVectors v,
                                                       int nrhs, int group, int maxk, int up, int root) {
  extern __shared__ __align__(16) unsigned char smem[];
  cplx<double>* in = (cplx<double>*)smem;   // [group][maxk]
  constexpr int kSlices = 256 / Rows, kSpan = Rows > kWave ? Rows : kWave, kParts = 256 / kSpan;
  __shared__ cplx<double> red[kNdRhsGroup][kParts][Rows];
  const NdNode nd = nodes[first + blockIdx.y];
  const int m = nd.s + nd.b, R = up ? nd.b : nd.s, K = up ? nd.s : m;
  const int tid = threadIdx.x, r = tid % Rows, sl = tid / Rows, row0 = blockIdx.x * Rows;
  if (row0 >= R) return;
  const int row = min(row0 + r, R - 1);
  const double* __restrict__ M = fac + (up ? nd.up : nd.down) + row;
  auto load = [&](double (&mk)[Cols], int k0) {
#pragma unroll
    for (int u = 0; u < Cols; ++u) mk[u] = M[(long long)min(k0 + u * kSlices, K - 1) * R];
  };
  for (int q0 = 0; q0 < nrhs; q0 += group) {
    const int ng = min(group, nrhs - q0);
    double m0[Cols], m1[Cols];
    load(m0, sl);
    for (int q = 0; q < ng; ++q) {
      for (int k = tid; k < K; k += 256) {
        const int rhs = q0 + q;
        cplx<double> x;
        if (up || (root && k < nd.s)) x = nd_received(nd, idx, cpos, nidx, v, rhs, k);
        else if (k < nd.s) x = v.y[rhs * v.ystride + idx[nd.idx + k]];
        else x = v.x[rhs * v.xstride + idx[nd.idx + k]];
        in[q * maxk + k] = x;
        if (up && row0 == 0) v.y[rhs * v.ystride + idx[nd.idx + k]] = x;
      }
    }
    __syncthreads();
    cplx<double> acc[kNdRhsGroup];
#pragma unroll
    for (int q = 0; q < kNdRhsGroup; ++q) acc[q] = czero<double>();
    for (int base = 0; base < K; base += Cols * kSlices) {
      const int k0 = base + sl;
      if (base + Cols * kSlices < K) load(m1, k0 + Cols * kSlices);
#pragma unroll
      for (int u = 0; u < Cols; ++u) {
        const int k = k0 + u * kSlices;
        if (k < K) {
#pragma unroll
          for (int q = 0; q < kNdRhsGroup; ++q) {
            if (q < ng) {
              const cplx<double> x = in[q * maxk + k];
              acc[q].re = fma(m0[u], x.re, acc[q].re);
              acc[q].im = fma(m0[u], x.im, acc[q].im);
            }
          }
        }
      }
#pragma unroll
      for (int u = 0; u < Cols; ++u) m0[u] = m1[u];
    }
    // sum the slices: within each wave (lanes equal modulo Rows), then through LDS
#pragma unroll
    for (int q = 0; q < kNdRhsGroup; ++q) {
      if (q < ng) {
        if (Rows <= 32) acc[q] = cplx<double>{fold32(acc[q].re, acc[q].re), fold32(acc[q].im, acc[q].im)};
        if (Rows <= 16) acc[q] = cplx<double>{fold16(acc[q].re, acc[q].re), fold16(acc[q].im, acc[q].im)};
        if (Rows <= 8) {
          acc[q].re += dpp_f64<kDppRowRor8>(acc[q].re);
          acc[q].im += dpp_f64<kDppRowRor8>(acc[q].im);
        }
        if (tid % kSpan < Rows) red[q][tid / kSpan][r] = acc[q];
      }
    }
    __syncthreads();
    for (int e = tid; e < ng * Rows; e += 256) {
      const int q = e / Rows, rr = e % Rows, orow = row0 + rr, rhs = q0 + q;
      if (orow < R) {
        cplx<double> t = red[q][0][rr];
#pragma unroll
        for (int j = 1; j < kParts; ++j) t = t + red[q][j][rr];
        if (up) v.g[rhs * v.gstride + nd.g + orow] = t + nd_received(nd, idx, cpos, nidx, v, rhs, nd.s + orow);
        else v.x[rhs * v.xstride + idx[nd.idx + orow]] = t;
      }
    }
    __syncthreads();
  }
}

// r = b - E_0 x over the coarse grid.
__global__ void __launch_bounds__(256) nd_refine_residual_kernel(const double* __restrict__ E0c, int n,
                                                                 const cplx<double>* __restrict__ b,
                                                                 const cplx<double>* __restrict__ x, long long stride,
                                                                 cplx<double>* __restrict__ r, long long rstride) {
  const int c = blockIdx.x * 256 + threadIdx.x, rhs = blockIdx.y;
  if (c >= n * n) return;
  const int cx = c % n, cy = c / n;
  cplx<double> acc = b[rhs * stride + c];
#pragma unroll
  for (int o = 0; o < 9; ++o) {
    const int dx = o % 3 - 1, dy = o / 3 - 1;
    if (cx + dx < 0 || cx + dx >= n || cy + dy < 0 || cy + dy >= n) continue;
    const double e = E0c[(long long)c * 9 + o];
    const cplx<double> v = x[rhs * stride + c + dy * n + dx];
    acc.re = fma(-e, v.re, acc.re);
    acc.im = fma(-e, v.im, acc.im);
  }
  r[rhs * rstride + c] = acc;
}

__global__ void __launch_bounds__(256) nd_add_kernel(cplx<double>* __restrict__ x, long long xstride,
                                                     const cplx<double>* __restrict__ d, long long dstride, int n) {
  const int c = blockIdx.x * 256 + threadIdx.x, rhs = blockIdx.y;
  if (c < n) x[rhs * xstride + c] = x[rhs * xstride + c] + d[rhs * dstride + c];
}

// Per workgroup |x|^2 and |d|^2.
__global__ void __launch_bounds__(256) nd_norms_kernel(const cplx<double>* __restrict__ x,
                                                       const cplx<double>* __restrict__ d, long long n,
                                                       double* __restrict__ out) {
  double a = 0.0, b = 0.0;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < n; e += gridDim.x * 256ll) {
    a += cabs2(x[e]);
    b += cabs2(d[e]);
  }
  a = wave_sum(a);
  b = wave_sum(b);
  __shared__ double sh[2][256 / kWave];
  if (threadIdx.x % kWave == 0) { sh[0][threadIdx.x / kWave] = a; sh[1][threadIdx.x / kWave] = b; }
  __syncthreads();
  if (threadIdx.x < 2) {
    double r = 0.0;
    for (int w = 0; w < 256 / kWave; ++w) r += sh[threadIdx.x][w];
    out[2 * blockIdx.x + threadIdx.x] = r;
  }
}

constexpr int kNdLds = 96 * 1024;      // LDS for the gathered vectors of the solve kernel
constexpr int kMaxGridY = 65535;
constexpr int kNdNormBlocks = 32;

// The tree of boxes of an n x n grid and what the solve and the set-up need to know of it.
struct NdPlan {
  std::vector<NdNode> nodes;
  std::vector<NdLevel> levels;
  std::vector<int> idx, cpos;     // cpos: kNdChildren arrays of idx's length
  long long nfac = 0, glen = 0;
  std::vector<long long> front_len, inv_len;   // per depth
  std::vector<int> panel_len;
};

NdPlan nd_plan(int n) {
  struct Box { int x0, x1, y0, y1; };
  NdPlan P;
  std::vector<Box> boxes{{0, n, 0, n}}, next;
  std::vector<int> where((size_t)n * n, -1);   // front position of a grid node in the box at hand
  int first = 0;
  while (!boxes.empty()) {
    NdLevel lv{first, (int)boxes.size(), 0, 0, 0};
    long long fl = 0, il = 0;
    int pl = 0;
    next.clear();
    for (const Box& B : boxes) {
      NdNode nd{};
      nd.idx = (int)P.idx.size();
      nd.kid = first + lv.count + (int)next.size();
      const int w = B.x1 - B.x0, h = B.y1 - B.y0;
      auto add = [&](int x, int y) { P.idx.push_back(y * n + x); };
      const bool cutx = w > kNdLeaf, cuty = h > kNdLeaf;
      const int cx = (B.x0 + B.x1) / 2, cy = (B.y0 + B.y1) / 2;
      for (int y = B.y0; y < B.y1; ++y)
        for (int x = B.x0; x < B.x1; ++x)
          if ((!cutx && !cuty) || (cutx && x == cx) || (cuty && y == cy)) add(x, y);
      nd.s = (int)P.idx.size() - nd.idx;
      for (int y = B.y0 - 1; y <= B.y1; ++y)
        for (int x = B.x0 - 1; x <= B.x1; ++x)
          if (x >= 0 && x < n && y >= 0 && y < n && (x < B.x0 || x >= B.x1 || y < B.y0 || y >= B.y1)) add(x, y);
      nd.b = (int)P.idx.size() - nd.idx - nd.s;
      if (cutx || cuty) {
        const int xs[2][2] = {{B.x0, cutx ? cx : B.x1}, {cx + 1, B.x1}};
        const int ys[2][2] = {{B.y0, cuty ? cy : B.y1}, {cy + 1, B.y1}};
        for (int b = 0; b < (cuty ? 2 : 1); ++b)
          for (int a = 0; a < (cutx ? 2 : 1); ++a) next.push_back(Box{xs[a][0], xs[a][1], ys[b][0], ys[b][1]});
        nd.kids = first + lv.count + (int)next.size() - nd.kid;
      }
      const long long m = nd.s + nd.b;
      nd.g = (int)P.glen;
      P.glen += nd.b;
      nd.up = P.nfac;
      nd.down = nd.up + (long long)nd.s * nd.b;
      P.nfac = nd.down + (long long)nd.s * m;
      nd.front = fl;
      fl += m * m;
      nd.inv = il;
      il += (long long)nd.s * nd.s;
      nd.panel = pl;
      pl += nd.s;
      nd.steps = (nd.s + kNdPivot - 1) / kNdPivot;
      lv.max_s = std::max(lv.max_s, nd.s);
      lv.max_b = std::max(lv.max_b, nd.b);
      lv.steps = std::max(lv.steps, nd.steps);
      P.nodes.push_back(nd);
    }
    P.front_len.push_back(fl);
    P.inv_len.push_back(il);
    P.panel_len.push_back(pl);
    first += lv.count;
    P.levels.push_back(lv);
    boxes.swap(next);
  }
  const size_t len = P.idx.size();
  P.cpos.assign(kNdChildren * len, -1);
  for (const NdNode& nd : P.nodes) {
    if (!nd.kids) continue;
    for (int f = 0; f < nd.s + nd.b; ++f) where[P.idx[nd.idx + f]] = f;
    for (int c = 0; c < nd.kids; ++c) {
      const NdNode& kd = P.nodes[nd.kid + c];
      for (int j = 0; j < kd.b; ++j) P.cpos[c * len + nd.idx + where[P.idx[kd.idx + kd.s + j]]] = kd.g + j;
    }
  }
  return P;
}

}  // namespace

#define ND_TRY(x)                        \
  do {                                   \
    hipError_t e_ = (x);                 \
    if (e_ != hipSuccess) return e_;     \
  } while (0)

NdMemory::~NdMemory() {
  for (void* p : blocks) (void)hipFree(p);
}

hipError_t NdMemory::take(void** p, size_t bytes) {
  bytes = (std::max<size_t>(bytes, 1) + 255) & ~size_t(255);
  const bool shared = bytes <= kNdSmall;
  if (!shared || bytes > room) {
    void* q = nullptr;
    ND_TRY(hipMalloc(&q, shared ? kNdChunk : bytes));
    blocks.push_back(q);
    if (!shared) {
      *p = q;
      return hipSuccess;
    }
    chunk = (unsigned char*)q;
    room = kNdChunk;
  }
  *p = chunk;
  chunk += bytes;
  room -= bytes;
  return hipSuccess;
}

hipError_t NestedDissection::setup(const double* E, int n, int nr, cplx<double>* vec, hipStream_t st) {
  E0c = E;
  nc = n;
  ncoarse = (long long)n * n;
  cv = vec;

  // ---- factor on the device: depth by depth, the smallest boxes first ----
  const NdPlan P = nd_plan(nc);
  levels = P.levels;
  nfac = P.nfac;
  glen = P.glen;
  nidx = (long long)P.idx.size();
  const size_t count = P.nodes.size();
  solve_bytes = 0;
  for (const NdNode& nd : P.nodes) {
    const long long m = nd.s + nd.b;
    // the solve matrices, and each vector entry read and written once per direction
    solve_bytes += 8 * (nd.s * m + (long long)nd.s * nd.b) + 16 * (2 * m + 2 * nd.s);
  }
  ND_TRY(memory.take(&fac, (size_t)nfac));
  // the plan in one copy: nodes, grid indices, child positions
  const size_t idx_at = sizeof(NdNode) * count, cpos_at = idx_at + sizeof(int) * P.idx.size();
  std::vector<unsigned char> plan(cpos_at + sizeof(int) * P.cpos.size());
  std::memcpy(plan.data(), P.nodes.data(), idx_at);
  std::memcpy(plan.data() + idx_at, P.idx.data(), cpos_at - idx_at);
  std::memcpy(plan.data() + cpos_at, P.cpos.data(), plan.size() - cpos_at);
  unsigned char* dplan = nullptr;
  ND_TRY(memory.take(&dplan, plan.size()));
  nodes = (NdNode*)dplan;
  idx = (int*)(dplan + idx_at);
  cpos = (int*)(dplan + cpos_at);
  ND_TRY(memory.take(&yv, (size_t)nr * ncoarse));
  ND_TRY(memory.take(&gv, (size_t)nr * std::max<long long>(glen, 1)));
  ND_TRY(memory.take(&rv, (size_t)nr * 2 * ncoarse));
  ND_TRY(hipMemcpyAsync(dplan, plan.data(), plan.size(), hipMemcpyHostToDevice, st));
  // the solve kernel's largest LDS request, before anything is captured
  for (const void* fn : {(const void*)nd_solve_kernel<64, 8>, (const void*)nd_solve_kernel<16, 8>, (const void*)nd_solve_kernel<8, 8>})
    ND_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kNdLds));
  // two depths of fronts are alive at a time; everything else is of one depth
  size_t len[2] = {1, 1}, ilen = 1, plen = 1, widest = 1;
  for (size_t d = 0; d < levels.size(); ++d) {
    len[d % 2] = std::max(len[d % 2], (size_t)P.front_len[d]);
    ilen = std::max(ilen, (size_t)P.inv_len[d]);
    plen = std::max(plen, (size_t)P.panel_len[d]);
    widest = std::max(widest, (size_t)levels[d].count);
  }
  NdMemory temp;
  double *front[2] = {nullptr, nullptr}, *X[3] = {nullptr, nullptr, nullptr}, *rows = nullptr, *cols = nullptr;
  double *dinv = nullptr, *dpiv = nullptr;
  for (int q = 0; q < 2; ++q) ND_TRY(temp.take(&front[q], len[q]));
  for (int q = 0; q < 3; ++q) ND_TRY(temp.take(&X[q], ilen));
  ND_TRY(temp.take(&rows, plen * kNdPivot));
  ND_TRY(temp.take(&cols, plen * kNdPivot));
  ND_TRY(temp.take(&dinv, widest * kNdPivot * kNdPivot));
  std::vector<double> out(count + 2 * kNdNormBlocks);   // the smallest pivots, then norms
  ND_TRY(temp.take(&dpiv, out.size()));
  for (int d = (int)levels.size() - 1; d >= 0; --d) {
    const NdLevel& lv = levels[d];
    double* F = front[d % 2];
    auto tiles = [](int v) { return (unsigned)std::max(1, (v + kNdTile - 1) / kNdTile); };
    const unsigned ts = tiles(lv.max_s), tb = tiles(lv.max_b);
    const int max_m = lv.max_s + lv.max_b;
    const unsigned spread = (unsigned)std::min<long long>(((long long)max_m * max_m + 255) / 256, 1024);
    for (int c0 = 0; c0 < lv.count; c0 += kMaxGridY) {   // (grid y is limited)
      const unsigned cnt = (unsigned)std::min(kMaxGridY, lv.count - c0);
      const NdNode* nds = nodes;
      const int at = lv.first + c0;
      hipLaunchKernelGGL(nd_front_kernel, dim3(spread, cnt), dim3(256), 0, st, nds, at, (const int*)idx,
                         (const int*)cpos, nidx, (const double*)E0c, nc, (const double*)front[(d + 1) % 2], F, X[0]);
      for (int t = 0; t < lv.steps; ++t) {
        hipLaunchKernelGGL(nd_pivot_kernel, dim3(cnt), dim3(256), 0, st, nds, at, t, (const double*)X[0], dinv, dpiv);
        hipLaunchKernelGGL(nd_panel_kernel, dim3(ts, cnt), dim3(256), 0, st, nds, at, t, (const double*)X[0],
                           (const double*)dinv, rows, cols);
        hipLaunchKernelGGL(nd_eliminate_kernel, dim3(ts * ts, cnt), dim3(256), 0, st, nds, at, t, X[0],
                           (const double*)rows, (const double*)cols);
      }
      const unsigned grid[4] = {ts * ts, ts * ts, ts * tb, tb * tb};
      for (int mode = 0; mode < (d > 0 ? 4 : 2); ++mode)
        hipLaunchKernelGGL(nd_product_kernel, dim3(grid[mode], cnt), dim3(256), 0, st, nds, at, mode, F,
                           (const double*)X[0], X[1], X[2], fac);
      hipLaunchKernelGGL(nd_extract_kernel, dim3(spread, cnt), dim3(256), 0, st, nds, at, (const double*)X[2], fac);
      ND_TRY(hipGetLastError());
    }
  }
  // error of a solve: the correction of one refinement, on a pseudo-random right-hand side
  refine = false;
  ND_TRY(launch_fill_hash(cv, ncoarse, 17081ull, st));
  ND_TRY(solve(1, st));
  ND_TRY(residual(1, st));
  ND_TRY(sweep(rv, 2 * ncoarse, rv + ncoarse, 2 * ncoarse, 1, st));
  hipLaunchKernelGGL(nd_norms_kernel, dim3(kNdNormBlocks), dim3(256), 0, st, (const cplx<double>*)(cv + ncoarse),
                     (const cplx<double>*)(rv + ncoarse), ncoarse, dpiv + count);
  ND_TRY(hipGetLastError());
  ND_TRY(hipMemcpyAsync(out.data(), dpiv, sizeof(double) * out.size(), hipMemcpyDeviceToHost, st));
  ND_TRY(hipStreamSynchronize(st));
  // smallest |pivot| over every pivot block; a non-finite one marks the factor unusable
  bool finite = true;
  min_pivot = INFINITY;
  for (size_t q = 0; q < count; ++q) {
    finite = finite && std::isfinite(out[q]);
    min_pivot = std::min(min_pivot, out[q]);
  }
  if (!finite) min_pivot = 0.0;
  if (!(min_pivot > 0.0)) return hipSuccess;
  double x2 = 0.0, d2 = 0.0;
  for (int q = 0; q < kNdNormBlocks; ++q) {
    x2 += out[count + 2 * q];
    d2 += out[count + 2 * q + 1];
  }
  solve_error = std::sqrt(d2 / x2);
  accurate = solve_error <= kNdRefuseAbove;   // (false for a NaN)
  refine = solve_error > kNdRefineAbove;
  if (refine) solve_bytes = 2 * solve_bytes + ncoarse * (9 * 8 + 3 * 16 + 3 * 16);
  return hipSuccess;
}

hipError_t NestedDissection::residual(int nr, hipStream_t st) {
  hipLaunchKernelGGL(nd_refine_residual_kernel, dim3((unsigned)((ncoarse + 255) / 256), (unsigned)nr), dim3(256), 0,
                     st, (const double*)E0c, nc, (const cplx<double>*)cv, (const cplx<double>*)(cv + ncoarse),
                     2 * ncoarse, rv, 2 * ncoarse);
  return hipGetLastError();
}

hipError_t NestedDissection::solve(int nr, hipStream_t st) {
  ND_TRY(sweep(cv, 2 * ncoarse, cv + ncoarse, 2 * ncoarse, nr, st));
  if (!refine) return hipSuccess;
  ND_TRY(residual(nr, st));
  ND_TRY(sweep(rv, 2 * ncoarse, rv + ncoarse, 2 * ncoarse, nr, st));
  hipLaunchKernelGGL(nd_add_kernel, dim3((unsigned)((ncoarse + 255) / 256), (unsigned)nr), dim3(256), 0, st,
                     cv + ncoarse, 2 * ncoarse, (const cplx<double>*)(rv + ncoarse), 2 * ncoarse, (int)ncoarse);
  return hipGetLastError();
}

// x = E_0^{-1} b, one pass up and one down.
hipError_t NestedDissection::sweep(const cplx<double>* b, long long bstride, cplx<double>* x, long long xstride, int nr,
                               hipStream_t st) {
  const NdVectors v{b, bstride, x, xstride, yv, ncoarse, gv, std::max<long long>(glen, 1)};
  auto launch = [&](const NdLevel& lv, int up, int root) -> hipError_t {
    const int R = up ? lv.max_b : lv.max_s, K = up ? lv.max_s : lv.max_s + lv.max_b;
    // right-hand sides per pass: as many as the gathered vectors leave LDS for
    const int group = std::max(1, std::min({kNdRhsGroup, nr, (int)(kNdLds / (K * sizeof(cplx<double>)))}));
    const size_t lds = (size_t)group * K * sizeof(cplx<double>);
    for (int c0 = 0; c0 < lv.count; c0 += kMaxGridY) {
      const unsigned cnt = (unsigned)std::min(kMaxGridY, lv.count - c0);
      // rows per workgroup: 64 while that gives every compute unit two workgroups, else 16 or 8 (more
      // column slices, shorter chains); every workgroup gathers its box's inputs, so 32 rows with all
      // columns in flight are slower at the deepest depth (25 -> 30 us at n = 317)
      auto go = [&](auto kernel, int rows) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((R + rows - 1) / rows), cnt), dim3(256), lds, st,
                           (const NdNode*)nodes, lv.first + c0, (const int*)idx, (const int*)cpos, nidx,
                           (const double*)fac, v, nr, group, K, up, root);
      };
      if ((long long)cnt * ((R + 63) / 64) >= 512) go(nd_solve_kernel<64, 8>, 64);
      else if ((long long)cnt * ((R + 15) / 16) >= 512) go(nd_solve_kernel<16, 8>, 16);
      else go(nd_solve_kernel<8, 8>, 8);
      ND_TRY(hipGetLastError());
    }
    return hipSuccess;
  };
  for (int d = (int)levels.size() - 1; d > 0; --d) ND_TRY(launch(levels[d], 1, 0));
  for (int d = 0; d < (int)levels.size(); ++d) ND_TRY(launch(levels[d], 0, d == 0));
  return hipSuccess;
}

}  // namespace ddh
