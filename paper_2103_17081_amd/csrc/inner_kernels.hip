// Batched inexact subdomain solves: GMRES on the deflated systems P_j B_j x = P_j f_j
// (Sec. 2, eq. 4; Sec. 3), all subdomains and right-hand sides in one launch.
//
// One workgroup carries one (subdomain, right-hand side) pair through its whole
// solve -- gather, deflated-operator applications, delayed-CGS2 Arnoldi with Givens
// rotations, its own convergence test, solution recovery, scatter -- so solves of
// uneven size and uneven iteration count run side by side without host round trips.
// Fine-level vectors are in the template precision T; the coarse solve is FP64.
//
// Per solve, with f = R_j r:
//   P f = f - B Z E^{-1} Z^T f,   reference norm ||P f||;
//   optional guess g accepted iff ||P f - P B g|| < ||P f||, else x0 = 0;
//   Arnoldi on the deflated operator P B with classical Gram-Schmidt applied twice in
//   the delayed form of Swirydowicz, Langou, Ananthan, Yang and Thomas (2020): the
//   operator is applied to the candidate u~_j before its second orthogonalisation, and
//   u~_j = V_j s + alpha_j v_j, so P B U~_k = V_{k+1} H_k with U~_k = V_k T_k (T upper
//   triangular, column j = (s, alpha_j));
//   stop when the least-squares residual estimate <= tol * ||P f||;
//   x = x0 + U~ y = x0 + V (T y),  u = x + Z E^{-1} Z^T (f - B x)   (so f - B u = P (f - B x));
//   the coarse vector of the recovery is assembled from those the solve already formed,
//   E^{-1} Z^T (f - B x) = E^{-1} Z^T f - E^{-1} Z^T B x0 - sum_i y_i E^{-1} Z^T B u~_i,
//   so it costs no deflated application of its own;
//   z(owned nodes of j) = u.
//
// Bound by latency: a launch lasts as long as its slowest solve, a chain of phases each a few
// thousand cycles long.  Slowest solve of the k = 200, N = 637, 16 x 16 workload (47 x 47 tile, 13
// iterations, complex128, 512 threads), us per iteration before and after the phases were
// reshaped: coarse solve 22.5 -> 10.4 (coarse.hpp, CoarseChain), dot and update sweeps 17.5 -> 11.2
// (next step's products formed in the update sweep, loads of the next node ahead of the work on
// this one), bookkeeping 5.0 -> 3.2 (one wave's lanes instead of one thread), stencils,
// restriction and prolongation 9.9 -> 8.3 (interior rows with three real coefficients, reciprocal
// instead of division for the node coordinates, factor loads issued meanwhile).  Launch, us:
// k = 200 complex128 765 -> 478, complex64 695 -> 446; k = 100, N = 160, 8 x 8 complex128 339 -> 214.
#include <algorithm>
#include <type_traits>

#include "coarse.hpp"
#include "kernels.hpp"
#include "stencil.hpp"

namespace ddh {

namespace {

__host__ __device__ constexpr size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

template <typename T>
struct Lds {
  cplx<T>* A;          // fine tile (stencil input)
  cplx<T>* B;          // fine tile (stencil output / working vector)
  cplx<T>* tab;        // 9 row classes x 7 coefficients
  cplx<T>* red;        // wave partial sums, (threads / wave) x stride
  cplx<T>* hT;         // update coefficients of the new basis vector (s / alpha); then T y
  cplx<T>* hU;         // update coefficients of the next candidate
  cplx<double>* sv;    // V_j^H u~_j, then |u~_j|^2
  cplx<double>* cv;    // V_j^H w, u~_j^H w, |w|^2
  cplx<double>* ct;    // coarse right-hand side
  cplx<double>* ca;    // coarse solution
  cplx<double>* lc;    // lower couplings of E staged for the coarse solve (3 per coarse node)
  cplx<double>* h;     // Hessenberg column (maxit + 2)
  cplx<double>* g;     // rotated right-hand side (maxit + 1)
  cplx<double>* sn;    // Givens sines (maxit)
  double* cs;          // Givens cosines (maxit)
  double* scal;        // 8 scalars
  int* ctrl;           // 4 ints
  cplx<double>* chain; // scratch of the coarse solve's narrow form
  int stride;          // maxit + 2
};

// Place of the coarse solve's scratch: tile A (rewritten by the prolongation), made large enough.  Tiles that would
// need more room for that (and the couplings' padding) than the coarse vectors save below take the products cv instead (free until the
// operator is applied), if those are long enough.  Such tiles run the narrow form only: a block row of more
// than 16 unknowns means at least 68 nodes and 17 coarse ones.
constexpr size_t kChainBytes = detail::kChainScratch * sizeof(cplx<double>);

template <typename T>
__host__ __device__ bool scratch_in_cv(int max_nj, int max_nc, int maxit) {
  const size_t tile = align16((size_t)max_nj * sizeof(cplx<T>));
  return tile + 2 * (size_t)max_nc * sizeof(cplx<double>) < kChainBytes + 16 && maxit + 2 >= detail::kChainScratch;
}
static_assert(2 * (kNarrowMx + 1) * 2 * sizeof(cplx<float>) + 2 * (kNarrowMx + 1) * sizeof(cplx<double>) >= kChainBytes + 16,
              "wider forms keep their scratch in tile A");

template <typename T>
__host__ __device__ size_t tile_a_bytes(int max_nj, int max_nc, int maxit) {
  const size_t tile = align16((size_t)max_nj * sizeof(cplx<T>));
  return tile >= kChainBytes || scratch_in_cv<T>(max_nj, max_nc, maxit) ? tile : kChainBytes;
}

// The coarse vectors and the sums' wave partials share their place: the ones live within an
// operator application, the others between two.
template <typename T>
__host__ __device__ size_t coarse_or_partials_bytes(int max_nc, int maxit, int nt) {
  const size_t coarse = align16(2 * (size_t)max_nc * sizeof(cplx<double>));
  const size_t partials = align16((size_t)(nt / kWave) * (maxit + 2) * sizeof(cplx<T>));
  return coarse > partials ? coarse : partials;
}

template <typename T>
__host__ __device__ size_t lds_bytes(int max_nj, int max_nc, int maxit, int nt) {
  const size_t s = (size_t)maxit + 2;
  size_t b = 0;
  b += tile_a_bytes<T>(max_nj, max_nc, maxit) + align16((size_t)max_nj * sizeof(cplx<T>));
  b += align16(kClasses * kStencilPts * sizeof(cplx<T>));
  b += coarse_or_partials_bytes<T>(max_nc, maxit, nt);
  b += 2 * align16(s * sizeof(cplx<T>));
  b += 2 * align16(s * sizeof(cplx<double>));
  b += align16(lower_entries(max_nc) * sizeof(cplx<double>));
  b += 3 * align16(s * sizeof(cplx<double>));
  b += align16(s * sizeof(double));
  b += align16(8 * sizeof(double)) + align16(4 * sizeof(int));
  return b;
}

template <typename T, int NT>
__device__ Lds<T> carve(unsigned char* base, int max_nj, int max_nc, int maxit) {
  Lds<T> L;
  const size_t s = (size_t)maxit + 2;
  L.stride = (int)s;
  size_t o = 0;
  auto take = [&](size_t bytes) { unsigned char* p = base + o; o += align16(bytes); return p; };
  L.A = (cplx<T>*)take(tile_a_bytes<T>(max_nj, max_nc, maxit));
  L.B = (cplx<T>*)take((size_t)max_nj * sizeof(cplx<T>));
  L.tab = (cplx<T>*)take(kClasses * kStencilPts * sizeof(cplx<T>));
  L.ct = (cplx<double>*)take(coarse_or_partials_bytes<T>(max_nc, maxit, NT));
  L.ca = L.ct + max_nc;
  L.red = (cplx<T>*)L.ct;
  L.hT = (cplx<T>*)take(s * sizeof(cplx<T>));
  L.hU = (cplx<T>*)take(s * sizeof(cplx<T>));
  L.sv = (cplx<double>*)take(s * sizeof(cplx<double>));
  L.cv = (cplx<double>*)take(s * sizeof(cplx<double>));
  L.lc = (cplx<double>*)take(lower_entries(max_nc) * sizeof(cplx<double>));
  L.h = (cplx<double>*)take(s * sizeof(cplx<double>));
  L.g = (cplx<double>*)take(s * sizeof(cplx<double>));
  L.sn = (cplx<double>*)take(s * sizeof(cplx<double>));
  L.cs = (double*)take(s * sizeof(double));
  L.scal = (double*)take(8 * sizeof(double));
  L.ctrl = (int*)take(4 * sizeof(int));
  L.chain = scratch_in_cv<T>(max_nj, max_nc, maxit) ? L.cv : (cplx<double>*)L.A;
  return L;
}

// `v` if `keep`, else 0 (a select, not a branch).
template <typename T>
__device__ __forceinline__ cplx<T> keep_or_zero(bool keep, cplx<T> v) {
  return cplx<T>{keep ? v.re : T(0), keep ? v.im : T(0)};
}

// out (=|-=) B_j in over the tile; no synchronisation.  Nodes inside the tile have every
// neighbour and the interior row's three real coefficients, held in registers; the nodes of the
// tile's edge (192 of 2303 for a 49 x 47 tile) are one more pass with their class's seven
// coefficients, where neighbours outside the tile are read at the node itself and multiplied
// by zero.
template <typename T, bool kSubtract>
__device__ __forceinline__ void apply_B(const SubDesc& d, const cplx<T>* tab, const cplx<T>* in, cplx<T>* out) {
  const int nx = d.nx, ny = d.ny, nj = nx * ny, tid = fresh_tid();
  const cplx<T>* mid = tab + kStencilPts * 4;
  const T cc = mid[kC].re, ce = mid[kE].re, cd = mid[kNE].re;
  for (int n = tid; n < nj; n += blockDim.x) {
    const int lj = row_of(n, d.inv_nx), li = n - lj * nx;
    if (li > 0 && li < nx - 1 && lj > 0 && lj < ny - 1) {
      const cplx<T>* x = in + n;
      const cplx<T> side = (x[-1] + x[1]) + (x[-nx] + x[nx]), diag = x[-nx - 1] + x[nx + 1], xc = x[0];
      const cplx<T> acc{fma(cc, xc.re, fma(ce, side.re, cd * diag.re)), fma(cc, xc.im, fma(ce, side.im, cd * diag.im))};
      out[n] = kSubtract ? out[n] - acc : acc;
    }
  }
  const int edge = 2 * (nx + ny) - 4;
  for (int m = tid; m < edge; m += blockDim.x) {
    const int q = m - 2 * nx;
    const int li = q >= 0 ? (q & 1) * (nx - 1) : (m < nx ? m : m - nx);
    const int lj = q >= 0 ? 1 + (q >> 1) : (m < nx ? 0 : ny - 1);
    const int n = lj * nx + li;
    const cplx<T>* c = tab + kStencilPts * node_class(d.i0 + li, d.j0 + lj, d.ax, d.bx, d.ay, d.by);
    const bool hw = li > 0, he = li < nx - 1, hs = lj > 0, hn = lj < ny - 1;
    const cplx<T> xc = in[n];
    const cplx<T> xw = keep_or_zero(hw, in[hw ? n - 1 : n]);
    const cplx<T> xe = keep_or_zero(he, in[he ? n + 1 : n]);
    const cplx<T> xs = keep_or_zero(hs, in[hs ? n - nx : n]);
    const cplx<T> xsw = keep_or_zero(hs && hw, in[hs && hw ? n - nx - 1 : n]);
    const cplx<T> xn = keep_or_zero(hn, in[hn ? n + nx : n]);
    const cplx<T> xne = keep_or_zero(hn && he, in[hn && he ? n + nx + 1 : n]);
    cplx<T> acc = c[kC] * xc;
    acc = cfma(c[kW], xw, acc);
    acc = cfma(c[kE], xe, acc);
    acc = cfma(c[kS], xs, acc);
    acc = cfma(c[kSW], xsw, acc);
    acc = cfma(c[kN], xn, acc);
    acc = cfma(c[kNE], xne, acc);
    out[n] = kSubtract ? out[n] - acc : acc;
  }
}

// t = Z^T v, accumulated in double.  With `padded`, t is a coarse-solve LDS array and
// its entries from mx * my up to the solve length ncp are set to 0.
template <typename T>
__device__ __forceinline__ void restrict_to(const SubDesc& d, const cplx<T>* v, cplx<double>* t,
                                            bool padded = true) {
  const int nc = d.mx * d.my;
  if (d.defl != kLinear) {
    const int nout = padded ? d.ncp : nc;
    for (int c = fresh_tid(); c < nout; c += blockDim.x) {
      cplx<double> acc = czero<double>();
      if (c < nc) {
        const int cy = row_of(c, d.inv_mx), cx = c - cy * d.mx;
        for (int py = max(2 * cy - 1, 0); py <= 2 * cy + 3 && py < d.ny; ++py) {
          const double wy = zweight_kind(kBezier, py, cy);
          for (int px = max(2 * cx - 1, 0); px <= 2 * cx + 3 && px < d.nx; ++px)
            acc = acc + (wy * zweight_kind(kBezier, px, cx)) * ccast<double>(v[py * d.nx + px]);
        }
      }
      t[c] = acc;
    }
    return;
  }
  // fine rows/columns 2c, 2c+1, 2c+2 with weights 1/2, 1, 1/2; only 2c+2 can fall outside
  // the tile, and is then read at 2c+1 with weight 0
  for (int c = fresh_tid(); c < nc; c += blockDim.x) {
    const int cy = row_of(c, d.inv_mx), cx = c - cy * d.mx;
    const bool xin = 2 * cx + 2 < d.nx, yin = 2 * cy + 2 < d.ny;
    const int px[3] = {2 * cx, 2 * cx + 1, xin ? 2 * cx + 2 : 2 * cx + 1};
    const int py[3] = {2 * cy, 2 * cy + 1, yin ? 2 * cy + 2 : 2 * cy + 1};
    const double wx[3] = {0.5, 1.0, xin ? 0.5 : 0.0};
    const double wy[3] = {0.5, 1.0, yin ? 0.5 : 0.0};
    cplx<T> vv[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int e = 0; e < 3; ++e) vv[b][e] = v[py[b] * d.nx + px[e]];
    cplx<double> acc = czero<double>();
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int e = 0; e < 3; ++e) acc = acc + (wy[b] * wx[e]) * ccast<double>(vv[b][e]);
    t[c] = acc;
  }
}

// Z y at fine node (li, lj).
__device__ __forceinline__ cplx<double> prolong_at(const SubDesc& d, const cplx<double>* y, int li, int lj) {
  if (d.defl != kLinear) {
    // coarse nodes within distance 2 of the fine node: c in [(i - 3) / 2, (i + 1) / 2]
    const int ca = (li - 3) >> 1, cb = (lj - 3) >> 1;
    cplx<double> acc = czero<double>();
#pragma unroll
    for (int b = cb; b <= cb + 2; ++b) {
      if (b < 0 || b >= d.my) continue;
      const double wy = zweight_kind(kBezier, lj, b);
#pragma unroll
      for (int a2 = ca; a2 <= ca + 2; ++a2) {
        if (a2 < 0 || a2 >= d.mx) continue;
        acc = acc + (wy * zweight_kind(kBezier, li, a2)) * y[b * d.mx + a2];
      }
    }
    return acc;
  }
  // coarse nodes (li - 1) >> 1 and the next one per direction: weights 1 and 0 on a coarse line,
  // 1/2 and 1/2 between two; one outside the coarse grid is read at a valid node with weight 0
  const int ca = (li - 1) >> 1, cb = (lj - 1) >> 1;
  const bool x0 = ca >= 0, x1 = ca + 1 < d.mx, y0 = cb >= 0, y1 = cb + 1 < d.my;
  const double wx0 = x0 ? ((li & 1) ? 1.0 : 0.5) : 0.0, wx1 = x1 && !(li & 1) ? 0.5 : 0.0;
  const double wy0 = y0 ? ((lj & 1) ? 1.0 : 0.5) : 0.0, wy1 = y1 && !(lj & 1) ? 0.5 : 0.0;
  const int ex0 = x0 ? ca : 0, ex1 = x1 ? ca + 1 : 0;
  const cplx<double>* r0 = y + (y0 ? cb : 0) * d.mx;
  const cplx<double>* r1 = y + (y1 ? cb + 1 : 0) * d.mx;
  const cplx<double> v00 = r0[ex0], v01 = r0[ex1], v10 = r1[ex0], v11 = r1[ex1];
  const double w00 = wy0 * wx0, w01 = wy0 * wx1, w10 = wy1 * wx0, w11 = wy1 * wx1;
  return cplx<double>{fma(w00, v00.re, fma(w01, v01.re, fma(w10, v10.re, w11 * v11.re))),
                      fma(w00, v00.im, fma(w01, v01.im, fma(w10, v10.im, w11 * v11.im)))};
}

template <typename T>
__device__ __forceinline__ void prolong_to(const SubDesc& d, const cplx<double>* y, cplx<T>* v) {
  const int nx = d.nx, nj = nx * d.ny;
  for (int n = fresh_tid(); n < nj; n += blockDim.x) {
    const int lj = row_of(n, d.inv_nx), li = n - lj * nx;
    v[n] = ccast<T>(prolong_at(d, y, li, lj));
  }
}

// B := P v with v = B_j A if `apply`, else tile B itself; P v = v - B_j Z E^{-1} Z^T v (tile A is
// overwritten); E^{-1} Z^T v goes to `keep`, if given.  The coarse solve's factor loads are under
// way while v is formed and restricted.
template <typename T, int NT, int Kind>
__device__ __forceinline__ void deflated_op(const SubDesc& d, const cplx<double>* fac, Lds<T>& L, bool apply,
                                            cplx<double>* keep) {
  cplx<double>* scratch = Kind == kCoarseNarrow ? L.chain : reinterpret_cast<cplx<double>*>(L.A);
  coarse_solve<NT, Kind>(d, fac, L.lc, L.ct, L.ca, scratch, [&]() {
    if (apply) {
      apply_B<T, false>(d, L.tab, L.A, L.B);
      lds_barrier();
    }
    restrict_to(d, L.B, L.ct);
    lds_barrier();
  });
  prolong_to(d, L.ca, L.A);
  if (keep)
    for (int e = fresh_tid(); e < d.ncp; e += NT) keep[e] = L.ca[e];
  lds_barrier();
  apply_B<T, true>(d, L.tab, L.A, L.B);
  lds_barrier();
}

// Workgroup sum of a real partial; every thread gets the total.
template <typename T, int NT>
__device__ __forceinline__ double block_sum(T part, Lds<T>& L) {
  part = wave_total(part);
  const int tid = fresh_tid(), lane = tid % kWave, wave = tid / kWave;
  lds_barrier();
  if (lane == kWave - 1) L.red[wave].re = part;
  lds_barrier();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) s += (double)L.red[w].re;
  lds_barrier();
  return s;
}

template <int NT>
__device__ __forceinline__ double block_sum_f64(double part, double* red) {
  part = wave_total(part);
  const int tid = fresh_tid(), lane = tid % kWave, wave = tid / kWave;
  lds_barrier();
  if (lane == kWave - 1) red[wave] = part;
  lds_barrier();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) s += red[w];
  lds_barrier();
  return s;
}

template <typename T, int NT>
__device__ __forceinline__ double tile_norm(const SubDesc& d, const cplx<T>* v, Lds<T>& L) {
  const int nj = d.nx * d.ny;
  T p = T(0);
  for (int n = fresh_tid(); n < nj; n += NT) p += cabs2(v[n]);
  return sqrt(block_sum<T, NT>(p, L));
}

// ---- sweeps over the basis ------------------------------------------------------------
// Thread tid owns nodes tid, tid + NT, ... of the tile, and of every basis vector.  A sweep is bound
// by the latency of the basis loads, so a thread issues the loads of its next node before it
// works on the current one: `load(buf, n)` issues one node's loads, `use(buf, n, valid)` works on
// them, `put(n)` stores the results, after the next loads were issued.  Every path issues the
// same number of loads (past the end those of sweep_node, whose results are dropped): the
// wait before `use` then covers that node's loads only.  Waves past the end have nothing to do.
template <typename T, int Count>
struct SweepBuf {
  cplx<T> v[Count > 0 ? Count : 1], u;
};

template <typename T, int NT, int Count, typename Load, typename Use, typename Put>
__device__ __forceinline__ void sweep_nodes(int nj, Load load, Use use, Put put) {
  const int tid = fresh_tid(), steps = (nj + NT - 1) / NT;
  if (__builtin_amdgcn_readfirstlane(tid) >= nj) return;
  SweepBuf<T, Count> b0, b1;
  load(b0, sweep_node(tid, tid, nj));
  for (int e = 0; e + 1 < steps; e += 2) {
    const int n0 = tid + e * NT, n1 = n0 + NT;
    load(b1, sweep_node(n1, tid, nj));
    use(b0, n0, true);
    load(b0, sweep_node(n1 + NT, tid, nj));
    put(n0);
    use(b1, sweep_node(n1, tid, nj), n1 < nj);
    if (n1 < nj) put(n1);
  }
  if (steps & 1) {
    const int n = tid + (steps - 1) * NT;
    use(b0, sweep_node(n, tid, nj), n < nj);
    if (n < nj) put(n);
  }
}

// Vectors a sweep takes at a time: two nodes' entries and the accumulators fit in registers.
template <typename T>
constexpr int kSweepVecs = sizeof(T) == 4 ? 16 : 8;

// f(std::integral_constant<int, G>) with G = ceil(count / 4), count <= kSweepVecs<T>: the sweeps are
// compiled for whole groups of 4 vectors.
template <typename T, typename F>
__device__ __forceinline__ void for_groups(int count, F f) {
  const int g = (count + 3) / 4;
  if (g <= 1) f(std::integral_constant<int, 1>{});
  else if (kSweepVecs<T> == 8 || g == 2) f(std::integral_constant<int, 2>{});
  else if constexpr (kSweepVecs<T> > 8) {
    if (g == 3) f(std::integral_constant<int, 3>{});
    else f(std::integral_constant<int, 4>{});
  }
}

// Wave partials of the complex sums a and b to red[0] and red[1] of this wave.
template <typename T>
__device__ __forceinline__ void store_totals2(cplx<T> a, cplx<T> b, bool second, cplx<T>* red) {
  const T s = wave_totals4(a.re, a.im, b.re, b.im);   // rows: a.re, b.re, a.im, b.im
  const int lane = fresh_tid() % kWave, row = lane / 16;
  if (lane % 16 == 0 && (second || (row & 1) == 0)) reinterpret_cast<T*>(red)[2 * (row & 1) + (row >> 1)] = s;
}

// Gram-Schmidt coefficients against V[k0..k]: red[w * S + i] = wave w's partial of
// conj(V_i) . B for k0 <= i <= k, and red[w * S + k + 1] = wave w's partial of |B|^2 when
// with_norm.
template <typename T, int NT>
__device__ __forceinline__ void basis_dots(const cplx<T>* V, int nj, int k0, int k, const cplx<T>* B,
                                           cplx<T>* red, int S, bool with_norm) {
  const int tid = fresh_tid(), lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (int i0 = k0; i0 <= k; i0 += kSweepVecs<T>) {
    const cplx<T>* Vi = V + (long long)i0 * nj;
    const int last = min(k - i0, kSweepVecs<T> - 1);
    for_groups<T>(last + 1, [&](auto groups) {
      constexpr int C = 4 * decltype(groups)::value;
      cplx<T> acc[C];
#pragma unroll
      for (int q = 0; q < C; ++q) acc[q] = czero<T>();
      sweep_nodes<T, NT, C>(
          nj,
          [&](SweepBuf<T, C>& b, int n) {
#pragma unroll
            for (int q = 0; q < C; ++q) b.v[q] = Vi[(long long)min(q, last) * nj + n];
          },
          [&](const SweepBuf<T, C>& b, int n, bool valid) {
            const cplx<T> w = keep_or_zero(valid, B[n]);
#pragma unroll
            for (int q = 0; q < C; ++q) acc[q] = acc[q] + cmulc(b.v[q], w);
          },
          [](int) {});
#pragma unroll
      for (int q = 0; q < C; q += 2)
        if (q <= last) store_totals2(acc[q], acc[q + 1], q + 1 <= last, red + wave * S + i0 + q);
    });
  }
  if (with_norm) {
    T q = T(0);
    for (int n = tid; n < nj; n += NT) q += cabs2(B[n]);
    q = wave_total(q);
    if (lane == kWave - 1) red[wave * S + k + 1] = cplx<T>{q, T(0)};
  }
}

// B[n] += sum_{i < cnt} V_i[n] c_i over the tile.
template <typename T, int NT>
__device__ __forceinline__ void basis_combine(const cplx<T>* V, int nj, int cnt, const cplx<T>* c, cplx<T>* B) {
  for (int i0 = 0; i0 < cnt; i0 += kSweepVecs<T>) {
    const cplx<T>* Vi = V + (long long)i0 * nj;
    const int last = min(cnt - 1 - i0, kSweepVecs<T> - 1);
    for_groups<T>(last + 1, [&](auto groups) {
      constexpr int C = 4 * decltype(groups)::value;
      cplx<T> acc;
      sweep_nodes<T, NT, C>(
          nj,
          [&](SweepBuf<T, C>& b, int n) {
#pragma unroll
            for (int q = 0; q < C; ++q) b.v[q] = Vi[(long long)min(q, last) * nj + n];
          },
          [&](const SweepBuf<T, C>& b, int n, bool) {
            detail::wave_lds_order();   // the coefficients stay in LDS between nodes
            acc = B[n];
#pragma unroll
            for (int q = 0; q < C; ++q)
              if (q <= last) acc = acc + b.v[q] * c[i0 + q];
          },
          [&](int n) { B[n] = acc; });
    });
  }
}

// Delayed-CGS2 update sweep: with u = u~_j in slot j of V and w in LDS, at every node
//   v_j      = u / alpha - sum_{i<j} V_i ca_i              (written to slot j, over u)
//   u~_{j+1} = (w - sum_{i<j} V_i cb_i - u e) / gamma      (written to slot j + 1 and the tile)
// and, with the basis entries of the node still in registers, the next step's products
// V_i^H u~_{j+1} for the first kSweepVecs<T> vectors and v_j, and |u~_{j+1}|^2: these cost no sweep
// of their own (the later vectors of a long basis do).  Wave partials go to red[wave * S + i],
// i <= j + 1.
template <typename T, int NT>
__device__ __forceinline__ void basis_update_dots(cplx<T>* V, int nj, int j, const cplx<T>* ca, const cplx<T>* cb,
                                                  T inv_alpha, cplx<T> e, T inv_gamma, const cplx<T>* w,
                                                  cplx<T>* tile, cplx<T>* red, int S) {
  cplx<T>* Vj = V + (long long)j * nj;
  cplx<T>* Vn = Vj + nj;
  const int wave = __builtin_amdgcn_readfirstlane(fresh_tid() / kWave), head = min(j, kSweepVecs<T>);
  for_groups<T>(head, [&](auto groups) {
    constexpr int C = 4 * decltype(groups)::value;
    cplx<T> dot[C], dot_j = czero<T>(), un, vj;
    T nu = T(0);
#pragma unroll
    for (int q = 0; q < C; ++q) dot[q] = czero<T>();
    sweep_nodes<T, NT, C>(
        nj,
        [&](SweepBuf<T, C>& b, int n) {
          b.u = Vj[n];
#pragma unroll
          for (int q = 0; q < C; ++q) b.v[q] = V[(long long)max(min(q, head - 1), 0) * nj + n];
        },
        [&](const SweepBuf<T, C>& b, int n, bool valid) {
          detail::wave_lds_order();   // the coefficients stay in LDS between nodes
          cplx<T> aa = czero<T>(), ab = czero<T>();
#pragma unroll
          for (int q = 0; q < C; ++q) {
            if (q < head) {
              aa = cfma(b.v[q], ca[q], aa);
              ab = cfma(b.v[q], cb[q], ab);
            }
          }
          if constexpr (C == kSweepVecs<T>) {
            for (int i0 = kSweepVecs<T>; i0 < j; i0 += 4) {
              cplx<T> vl[4];
#pragma unroll
              for (int q = 0; q < 4; ++q) vl[q] = V[(long long)min(i0 + q, j - 1) * nj + n];
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                if (i0 + q < j) {
                  aa = cfma(vl[q], ca[i0 + q], aa);
                  ab = cfma(vl[q], cb[i0 + q], ab);
                }
              }
            }
          }
          un = keep_or_zero(valid, inv_gamma * (w[n] - ab - b.u * e));
          vj = inv_alpha * b.u - aa;
#pragma unroll
          for (int q = 0; q < C; ++q)
            if (q < head) dot[q] = dot[q] + cmulc(b.v[q], un);
          dot_j = dot_j + cmulc(vj, un);
          nu += cabs2(un);
        },
        [&](int n) {
          Vj[n] = vj;
          Vn[n] = un;
          tile[n] = un;
        });
#pragma unroll
    for (int q = 0; q < C; q += 2)
      if (q < head) store_totals2(dot[q], dot[q + 1], q + 1 < head, red + wave * S + q);
    store_totals2(dot_j, cplx<T>{nu, T(0)}, true, red + wave * S + j);
  });
  // every thread reads back only what it wrote
  if (j > kSweepVecs<T>) basis_dots<T, NT>(V, nj, kSweepVecs<T>, j - 1, tile, red, S, false);
}

template <typename T>
__host__ __device__ constexpr double breakdown_eps() { return sizeof(T) == 4 ? 4e-6 : 1e-14; }

}  // namespace

// A value every lane holds alike (a workgroup sum read back from LDS), moved to scalar
// registers: the Krylov loop keeps such values live, and in vector registers they would
// push the coarse solve's factor ring into scratch.
__device__ __forceinline__ double uniform_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
  const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The same for an offset (64-bit products are formed in vector registers).
__device__ __forceinline__ long long uniform_i64(long long v) {
  const int lo = __builtin_amdgcn_readfirstlane((int)(v & 0xffffffffll));
  const int hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
  return ((long long)hi << 32) | (unsigned int)lo;
}

// A uniform offset, opaque to the compiler here (see fresh_tid).
__device__ __forceinline__ long long fresh_offset(long long v) {
  asm volatile("" : "+s"(v));
  return v;
}

constexpr int kBatch = 8;   // loads issued together in the small gathers below

// Lane q's value of v (q uniform).
__device__ __forceinline__ double lane_value(double v, int q) {
  const long long b = __double_as_longlong(v);
  return join_f64((unsigned)__builtin_amdgcn_readlane((int)(b & 0xffffffffll), q),
                  (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), q));
}

// Sum of the wave partials of one coefficient (waves S apart), in wave order.
template <typename T, int NT>
__device__ __forceinline__ cplx<double> sum_waves(const cplx<T>* red, int S) {
  cplx<double> s = czero<double>();
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) s = s + ccast<double>(red[w * S]);
  return s;
}

template <typename T, int NT, int Kind>
__device__ __forceinline__ void inner_solve(const InnerArgs<T>& a, unsigned char* smem) {
  const int sidx = __builtin_amdgcn_readfirstlane(a.order ? a.order[blockIdx.x] : (int)blockIdx.x);
  const int nsub = a.cs.nsub;
  const int rhs = sidx / nsub, sub = sidx - rhs * nsub;
  if (a.done && a.done[rhs]) return;
  SubDesc d = a.subs[sub];
  if constexpr (Kind != kCoarseGeneral) d.defl = kLinear;   // (what these kernels are launched for)
  Lds<T> L = carve<T, NT>(smem, a.max_nj, a.max_nc, a.maxit);
  const int tid = threadIdx.x;
  const int nx = d.nx, nj = d.nx * d.ny;
  const int maxit = a.maxit;
  const long long fo = uniform_i64((long long)rhs * a.nfine + d.off);
  cplx<T>* F = a.F + fo;
  cplx<T>* V = a.V + uniform_i64(fo * (maxit + 1));
  // R factor of the rotated Hessenberg matrix, then T (candidates in the orthonormal basis),
  // each maxit x maxit with column c at c * maxit
  cplx<double>* R = a.R + uniform_i64((long long)sidx * 2 * maxit * maxit);
  cplx<double>* Tm = R + (long long)maxit * maxit;
  // coarse vectors kept for the recovery: slot 0 E^{-1} Z^T f, slot 1 E^{-1} Z^T B x0, slot 2 + i
  // E^{-1} Z^T B u~_i
  cplx<double>* Sc = a.Sc + uniform_i64((long long)sidx * (maxit + 2) * a.max_nc);
  const int ldg = a.cs.n - 1;
  const long long jstep = a.jdev ? (long long)*a.jdev : 0;
  const cplx<double>* __restrict__ rin = a.r ? a.r + jstep * a.rslot : nullptr;
  cplx<double>* __restrict__ zout = a.z ? a.z + jstep * a.zslot : nullptr;

  build_class_table<T>(d.robin, a.cs.kh, a.cs.kh2, L.tab);
  stage_lower(d, a.Ec, L.lc);
  // Gather f = R_j r.  The local system is linear and its stopping test relative,
  // so it is solved for f / ||f|| (norm taken in FP64) and the solution rescaled:
  // local right-hand sides far from the sources are many orders of magnitude below
  // 1 and would lose precision, or underflow, in complex64.
  double fn2 = 0.0;
  for (int n = tid; n < nj; n += NT) {
    if (rin) {
      const int lj = row_of(n, d.inv_nx), li = n - lj * nx;
      fn2 += cabs2(rin[(long long)rhs * a.rstride + (long long)(d.j0 + lj - 1) * ldg + (d.i0 + li - 1)]);
    } else {
      fn2 += cabs2(ccast<double>(F[n]));
    }
  }
  const double fnorm = uniform_f64(sqrt(block_sum_f64<NT>(fn2, (double*)L.red)));
  const double fscale = uniform_f64(fnorm > 0.0 ? 1.0 / fnorm : 0.0);
  // F holds the scaled right-hand side when gathered here; a caller-supplied F is
  // left untouched and scaled on use (fmul).
  const T fmul = rin ? T(1) : T(fscale);
  for (int n = tid; n < nj; n += NT) {
    cplx<T> v;
    if (rin) {
      const int lj = row_of(n, d.inv_nx), li = n - lj * nx;
      v = ccast<T>(fscale * rin[(long long)rhs * a.rstride + (long long)(d.j0 + lj - 1) * ldg + (d.i0 + li - 1)]);
      F[n] = v;
    } else {
      v = fmul * F[n];
    }
    L.B[n] = v;
  }
  lds_barrier();
  // One pass of the loop below projects tile B (B := P B) and goes on from there, so the
  // coarse solve is compiled once: pass 1 forms P f, pass 2 P B g of an offered guess, the
  // others w = P B u~_j of the Krylov iteration.
  const bool guessed = a.guess || a.gtile;
  bool accepted = false, offered = false, converged = true;
  double ref = 0.0;
  int k = 0, stage = 0;      // stage 0: P f, 1: P B g, 2: Krylov
  const int S = L.stride;
  // Iteration j: (1) s = V_j^H u~_j, nu = |u~_j|^2 (formed by the previous update sweep), alpha =
  // sqrt(nu - |s|^2); column j-1 of H becomes final (tentative column + gamma_j s, subdiagonal
  // gamma_j alpha), is rotated, and the residual estimate decides convergence before the
  // operator is applied; (2) w = P B u~_j; (3) c = V_j^H w, mu = u~_j^H w, omega = |w|^2; tentative
  // column j: c and h_jj = (mu - s^H c) / alpha; gamma_{j+1} from Pythagoras (a scale only: the
  // next step's nu corrects it exactly); (4) one update sweep writes v_j and u~_{j+1}.
  int j = 0;
  bool apply = false;        // the first pass projects f itself
  while (true) {
    deflated_op<T, NT, Kind>(d, a.fac, L, apply, Sc + (long long)(stage < 2 ? stage : 2 + j) * a.max_nc);
    apply = true;
    const int tid = fresh_tid();
    if (stage < 2) {
      cplx<T>* W = a.W + fresh_offset(fo);
      cplx<T>* X = a.X + fresh_offset(fo);
      double beta;
      if (stage == 0) {
        ref = uniform_f64(tile_norm<T, NT>(d, L.B, L));
        if (!(ref > 0.0)) break;
        beta = ref;
        if (guessed) {
          offered = true;
          // the solve runs on f / ||f||: a packed guess is scaled by 1 / ||f||, a network
          // tile (scaled by sqrt(n_j) / ||f||) by 1 / sqrt(n_j)
          const cplx<T>* gs = a.guess ? a.guess + fo : nullptr;
          const float* gt = a.gtile ? a.gtile + (size_t)sidx * a.gT * a.gT * 2 : nullptr;
          const T gmul = gt ? T(1.0 / sqrt((double)fresh_offset(nj))) 
                             : T(__longlong_as_double(fresh_offset(__double_as_longlong(fscale))));
          for (int n = tid; n < nj; n += NT) {
            W[n] = L.B[n];
            cplx<T> gv;
            if (gt) {
              const int lj = row_of(n, d.inv_nx), li = n - lj * nx;
              const float* q = gt + ((size_t)lj * a.gT + li) * 2;
              gv = cplx<T>{gmul * T(q[0]), gmul * T(q[1])};
            } else {
              gv = gmul * gs[n];
            }
            L.A[n] = gv;
            X[n] = gv;
          }
          lds_barrier();
          stage = 1;
          continue;
        }
      } else {
        for (int n = tid; n < nj; n += NT) L.B[n] = W[n] - L.B[n];   // tile B held P B g
        lds_barrier();
        const double rn = tile_norm<T, NT>(d, L.B, L);
        accepted = __builtin_amdgcn_readfirstlane(rn < ref ? 1 : 0) != 0;
        if (!accepted) {
          for (int n = tid; n < nj; n += NT) L.B[n] = W[n];
          lds_barrier();
        }
        beta = accepted ? tile_norm<T, NT>(d, L.B, L) : ref;
      }
      stage = 2;
      converged = beta <= a.tol * ref;
      if (converged) break;
      // candidate u~_0 = r0 / beta in slot 0 and tile A
      const T inv = T(1.0 / beta);
      for (int n = tid; n < nj; n += NT) {
        const cplx<T> v = inv * L.B[n];
        V[n] = v;
        L.A[n] = v;
      }
      if (tid == 0) {
        L.g[0] = cplx<double>{beta, 0.0};
        L.ctrl[0] = 0;
      }
      basis_dots<T, NT>(V, nj, 0, -1, L.A, L.red, S, true);   // nu = |u~_0|^2
    } else {
      // tile B = w = P B u~_j (tile A overwritten)
      basis_dots<T, NT>(V, nj, 0, j, L.B, L.red, S, true);
      lds_barrier();
      if (tid < kWave) {
        // tentative column j and the coefficients of the update sweep, by one wave
        cplx<double> sTc = czero<double>();
        double cc = 0.0;
        for (int i = tid; i <= j + 1; i += kWave) {
          const cplx<double> c = sum_waves<T, NT>(L.red + i, S);
          L.cv[i] = c;
          if (i < j) {
            sTc = sTc + cmulc(L.sv[i], c);
            cc += cabs2(c);
          }
        }
        detail::wave_lds_order();
        sTc = cplx<double>{wave_total_all(sTc.re), wave_total_all(sTc.im)};
        cc = wave_total_all(cc);
        const double inv_alpha = L.scal[0], om = L.cv[j + 1].re;
        const cplx<double> hjj = inv_alpha * (L.cv[j] - sTc), e = inv_alpha * hjj;
        double g2 = om - cc - cabs2(hjj);
        const double gfloor = 1e-28 * (om > 0.0 ? om : 1.0);
        if (!(g2 > gfloor)) g2 = gfloor;
        const double gm = sqrt(g2);
        for (int i = tid; i <= j; i += kWave) {
          const cplx<double> c = L.cv[i];
          L.h[i] = cplx<double>{i < j ? c.re : hjj.re, i < j ? c.im : hjj.im};
          if (i < j) L.hU[i] = ccast<T>(c - L.sv[i] * e);
        }
        if (tid == 0) {
          L.scal[2] = sqrt(om > 0.0 ? om : 0.0);   // ||w||: breakdown scale of column j
          L.scal[3] = gm;
          L.scal[4] = 1.0 / gm;
          L.scal[6] = e.re;
          L.scal[7] = e.im;
        }
      }
      lds_barrier();
      const cplx<double> e{L.scal[6], L.scal[7]};
      basis_update_dots<T, NT>(V, nj, j, L.hT, L.hU, T(L.scal[0]), ccast<T>(e), T(L.scal[4]), L.B, L.A, L.red, S);
      ++j;
    }
    lds_barrier();
    if (tid < kWave) {
      // s, alpha, column j - 1 and its rotation, by one wave: lane i holds entry i (mod 64)
      double ss = 0.0;
      for (int i = tid; i <= j; i += kWave) {
        const cplx<double> v = sum_waves<T, NT>(L.red + i, S);
        L.sv[i] = v;
        if (i < j) ss += cabs2(v);
      }
      detail::wave_lds_order();
      ss = wave_total_all(ss);
      const double nu = L.sv[j].re;
      const double a2 = nu - ss, afloor = 1e-30 * (nu > 0.0 ? nu : 1.0);
      const double ac = a2 > afloor ? a2 : afloor, inv_alpha = rsqrt(ac), alpha = ac * inv_alpha;
      bool stop = false;
      if (j == 0) {
        if (tid == 0) L.g[0] = alpha * L.g[0];
      } else {
        const int c0 = j - 1;
        const double gm = L.scal[3];
        cplx<double>* col = L.h;
        for (int i = tid; i <= c0; i += kWave) col[i] = col[i] + gm * L.sv[i];
        detail::wave_lds_order();
        // rotations 0 .. c0-1: the entry carried down the column passes through registers, each lane
        // keeps the one its own rotation receives
        cplx<double> x = col[0];
        for (int b0 = 0; b0 < c0; b0 += kWave) {
          const int i = min(b0 + tid, c0 - 1), cnt = min(kWave, c0 - b0);
          const double cl = L.cs[i];
          const cplx<double> sl = L.sn[i], nl = col[i + 1];
          cplx<double> mine = czero<double>();
          for (int q = 0; q < cnt; ++q) {
            if (tid == q) mine = x;
            const double c = lane_value(cl, q);
            const cplx<double> sq{lane_value(sl.re, q), lane_value(sl.im, q)};
            const cplx<double> nq{lane_value(nl.re, q), lane_value(nl.im, q)};
            x = c * nq - cplx<double>{sq.re, -sq.im} * x;
          }
          if (tid < cnt) R[(long long)c0 * maxit + b0 + tid] = cl * mine + sl * nl;
        }
        const double hnext = gm * alpha;
        const double aa2 = cabs2(x);
        double c;
        cplx<double> sv, r;
        if (hnext == 0.0) {
          c = 1.0; sv = czero<double>(); r = x;
        } else if (aa2 == 0.0) {
          c = 0.0; sv = cplx<double>{1.0, 0.0}; r = cplx<double>{hnext, 0.0};
        } else {
          const double t2 = aa2 + hnext * hnext, it = rsqrt(t2), ia = rsqrt(aa2);
          const cplx<double> ph = ia * x;   // x / |x|
          c = (aa2 * ia) * it;
          sv = (hnext * it) * ph;
          r = (t2 * it) * ph;
        }
        const cplx<double> gk = L.g[c0];
        const cplx<double> gn = czero<double>() - cplx<double>{sv.re, -sv.im} * gk;
        const bool brk = hnext <= breakdown_eps<T>() * L.scal[2];
        stop = sqrt(cabs2(gn)) <= a.tol * ref || brk;
        if (tid == 0) {
          L.cs[c0] = c;
          L.sn[c0] = sv;
          R[(long long)c0 * maxit + c0] = r;
          L.g[c0 + 1] = gn;
          L.g[c0] = c * gk;
        }
      }
      if (tid == 0) {
        L.scal[0] = inv_alpha;
        L.ctrl[0] = stop ? 1 : 0;
      }
      if (!stop && j < maxit) {
        // column j of T and the update coefficients of v_j
        cplx<double>* Tc = Tm + (long long)j * maxit;
        for (int i = tid; i <= j; i += kWave) {
          const cplx<double> v = L.sv[i];
          Tc[i] = cplx<double>{i < j ? v.re : alpha, i < j ? v.im : 0.0};
          if (i < j) L.hT[i] = ccast<T>(inv_alpha * v);
        }
      }
    }
    lds_barrier();
    converged = __builtin_amdgcn_readfirstlane(L.ctrl[0]) != 0;
    if (converged || j == maxit) break;
  }
  const int lid = fresh_tid();
  if (ref > 0.0) {
    k = j;
    // y = R^{-1} g (upper triangular, k x k).  R is copied into the free tile A first when
    // it fits (all threads load it side by side), so the serial substitution reads LDS.
    const bool r_lds = (size_t)k * k * sizeof(cplx<double>) <= (size_t)a.max_nj * sizeof(cplx<T>);
    cplx<double>* Rl = reinterpret_cast<cplx<double>*>(L.A);
    __syncthreads();   // the global stores of R and T are visible to the workgroup
    if (r_lds) {
      for (int e = lid; e < k * k; e += NT) {
        const int j = e / k, i = e - j * k;
        if (i <= j) Rl[e] = R[(long long)j * maxit + i];
      }
      lds_barrier();
    }
    // column by column: lane l updates g_l with y_i as soon as it is known
    if (lid < kWave) {
      for (int i = lid; i < k; i += kWave) L.cv[i] = cinv(r_lds ? Rl[i * k + i] : R[(long long)i * maxit + i]);
      detail::wave_lds_order();
      for (int i = k - 1; i >= 0; --i) {
        const cplx<double> y = L.g[i] * L.cv[i];
        if (lid == 0) L.h[i] = y;
        for (int l = lid; l < i; l += kWave)
          L.g[l] = L.g[l] - (r_lds ? Rl[i * k + l] : R[(long long)i * maxit + l]) * y;
        detail::wave_lds_order();
      }
    }
    lds_barrier();
    // x coefficients in the orthonormal basis: T y (T upper triangular)
    for (int i = lid; i < k; i += NT) {
      cplx<double> acc = czero<double>();
      for (int l0 = i; l0 < k; l0 += kBatch) {
        cplx<double> tv[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) tv[q] = Tm[(long long)min(l0 + q, k - 1) * maxit + i];
#pragma unroll
        for (int q = 0; q < kBatch; ++q)
          if (l0 + q < k) acc = acc + tv[q] * L.h[l0 + q];
      }
      L.hT[i] = ccast<T>(acc);
    }
    lds_barrier();
  }
  // x = x0 + V y   (tile A)
  {
    const cplx<T>* X = a.X + fresh_offset(fo);
    for (int n = lid; n < nj; n += NT) L.A[n] = accepted ? X[n] : czero<T>();
  }
  basis_combine<T, NT>(V, nj, k, L.hT, L.A);
  lds_barrier();
  // recovery: u = x + Z E^{-1} Z^T (f - B x), from the kept coarse vectors (y_i in L.h)
  for (int e = lid; e < d.ncp; e += NT) {
    cplx<double> c = Sc[e];
    if (accepted) c = c - Sc[a.max_nc + e];
    for (int i0 = 0; i0 < k; i0 += kBatch) {
      cplx<double> sv[kBatch];
#pragma unroll
      for (int q = 0; q < kBatch; ++q) sv[q] = Sc[(long long)(2 + min(i0 + q, k - 1)) * a.max_nc + e];
#pragma unroll
      for (int q = 0; q < kBatch; ++q)
        if (i0 + q < k) c = c - L.h[i0 + q] * sv[q];
    }
    L.ca[e] = c;
  }
  lds_barrier();
  for (int n = lid; n < nj; n += NT) {
    const int lj = row_of(n, d.inv_nx), li = n - lj * nx;
    const cplx<T> u = L.A[n] + ccast<T>(prolong_at(d, L.ca, li, lj));
    if (a.U) a.U[fo + n] = ccast<T>(fnorm * ccast<double>(u));
    if (zout) {
      const int gi = d.i0 + li, gj = d.j0 + lj;
      if (gi >= d.oi0 && gi <= d.oi1 && gj >= d.oj0 && gj <= d.oj1) {
        const long long gidx = (long long)(gj - 1) * ldg + (gi - 1);
        const cplx<double> add = a.zadd ? a.zadd[(long long)rhs * a.ndof + gidx] : czero<double>();
        zout[(long long)rhs * a.zstride + gidx] = fnorm * ccast<double>(u) + add;
      }
    }
  }
  if (lid == 0) {
    if (a.iters) a.iters[sidx] = k;
    if (a.flags) a.flags[sidx] = (accepted ? 1 : 0) | (converged ? 0 : 2);
    if (a.counters) {
      atomicAdd(a.counters + 0, (unsigned long long)k);
      atomicAdd(a.counters + 1, 1ull);
      atomicMax(a.counters + 2, (unsigned long long)k);
      if (accepted) atomicAdd(a.counters + 3, 1ull);
      const unsigned long long s = sizeof(cplx<T>), nn = (unsigned long long)nj, kk = (unsigned long long)k;
      const unsigned long long own = (unsigned long long)(d.oi1 - d.oi0 + 1) * (d.oj1 - d.oj0 + 1);
      const unsigned long long fac_bytes = 16ull * (unsigned long long)coarse_solve_values(d);
      const unsigned long long ncp = (unsigned long long)d.ncp;
      // the update sweep of step j reads the vectors after its first kSweepVecs once more
      const unsigned long long late = k > kSweepVecs<T> + 1 ? (unsigned long long)(k - 1 - kSweepVecs<T>) : 0ull;
      unsigned long long bytes = 16ull * nn + (a.zadd ? 32ull : 16ull) * own +
                                 (kk + 1) * fac_bytes + 16ull * ncp * (2 * kk + 2) +
                                 (kk ? s * nn * (1 + 3 * kk + kk * (kk + 1) + late * (late + 1) / 2) : 0ull) + 2 * s * nn;
      if (offered) bytes += fac_bytes + (a.gtile ? 8ull : s) * nn + 3 * s * nn + 32ull * ncp;
      atomicAdd(a.counters + 4, bytes);
    }
  }
}

// One kernel per form of the coarse solve (CoarseKind).
template <typename T, int NT>
__global__ void __launch_bounds__(NT) inner_solve_kernel(InnerArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  inner_solve<T, NT, kCoarseChain>(a, smem);
}
template <typename T, int NT>
__global__ void __launch_bounds__(NT) inner_solve_narrow_kernel(InnerArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  inner_solve<T, NT, kCoarseNarrow>(a, smem);
}
template <typename T, int NT>
__global__ void __launch_bounds__(NT) inner_solve_general_kernel(InnerArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  inner_solve<T, NT, kCoarseGeneral>(a, smem);
}

template <typename T, int NT>
void (*inner_kernel(int kind))(InnerArgs<T>) {
  return kind == kCoarseNarrow ? inner_solve_narrow_kernel<T, NT>
                               : (kind == kCoarseChain ? inner_solve_kernel<T, NT> : inner_solve_general_kernel<T, NT>);
}

template <typename T>
size_t inner_lds_bytes(int max_nj, int max_nc, int maxit) {
  return std::max(lds_bytes<T>(max_nj, max_nc, maxit, kInnerThreads), lds_bytes<T>(max_nj, max_nc, maxit, 256));
}

template <typename T>
hipError_t launch_inner_solve(const InnerArgs<T>& a, hipStream_t st) {
  const int nblocks = a.cs.nsub * a.nrhs, nt = a.nt == 256 ? 256 : kInnerThreads;
  const size_t lds = lds_bytes<T>(a.max_nj, a.max_nc, a.maxit, nt);
  hipLaunchKernelGGL((nt == 256 ? inner_kernel<T, 256>(a.kind) : inner_kernel<T, kInnerThreads>(a.kind)), dim3(nblocks),
                     dim3(nt), lds, st, a);
  return hipGetLastError();
}

// ---- kernel-level operations on packed vectors ---------------------------------------

template <typename T>
__global__ void __launch_bounds__(kBlock) local_apply_kernel(const SubDesc* __restrict__ subs, Consts cs,
                                                              const cplx<T>* __restrict__ v,
                                                              cplx<T>* __restrict__ w) {
  extern __shared__ __align__(16) unsigned char smem[];
  const SubDesc d = subs[blockIdx.x];
  cplx<T>* tab = (cplx<T>*)smem;
  cplx<T>* tile = (cplx<T>*)(smem + align16(kClasses * kStencilPts * sizeof(cplx<T>)));
  build_class_table<T>(d.robin, cs.kh, cs.kh2, tab);
  const int nj = d.nx * d.ny;
  for (int n = threadIdx.x; n < nj; n += blockDim.x) tile[n] = v[d.off + n];
  __syncthreads();
  apply_B<T, false>(d, tab, tile, w + d.off);
}

template <typename T>
hipError_t launch_local_apply(const SubDesc* subs, int nsub, Consts cs, int, const cplx<T>* v, cplx<T>* w,
                              int max_nj, hipStream_t st) {
  const size_t lds = align16(kClasses * kStencilPts * sizeof(cplx<T>)) + (size_t)max_nj * sizeof(cplx<T>);
  hipLaunchKernelGGL(local_apply_kernel<T>, dim3(nsub), dim3(kBlock), lds, st, subs, cs, v, w);
  return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(kBlock) deflated_apply_kernel(const SubDesc* __restrict__ subs, Consts cs,
                                                                 const cplx<double>* __restrict__ fac,
                                                                 const cplx<double>* __restrict__ Ec,
                                                                 const cplx<T>* __restrict__ v,
                                                                 cplx<T>* __restrict__ w, int max_nj, int max_nc) {
  extern __shared__ __align__(16) unsigned char smem[];
  const SubDesc d = subs[blockIdx.x];
  Lds<T> L = carve<T, kBlock>(smem, max_nj, max_nc, 1);
  build_class_table<T>(d.robin, cs.kh, cs.kh2, L.tab);
  stage_lower(d, Ec, L.lc);
  const int nj = d.nx * d.ny;
  for (int n = threadIdx.x; n < nj; n += blockDim.x) L.A[n] = v[d.off + n];
  __syncthreads();
  const int kind = coarse_kind(d.defl, d.mx);
  if (kind == kCoarseNarrow) deflated_op<T, kBlock, kCoarseNarrow>(d, fac, L, true, nullptr);
  else if (kind == kCoarseChain) deflated_op<T, kBlock, kCoarseChain>(d, fac, L, true, nullptr);
  else deflated_op<T, kBlock, kCoarseGeneral>(d, fac, L, true, nullptr);
  for (int n = threadIdx.x; n < nj; n += blockDim.x) w[d.off + n] = L.B[n];
}

template <typename T>
hipError_t launch_deflated_apply(const SubDesc* subs, int nsub, Consts cs, int, const cplx<double>* fac,
                                 const cplx<double>* Ec, const cplx<T>* v, cplx<T>* w, int max_nj, int max_nc,
                                 hipStream_t st) {
  const size_t lds = lds_bytes<T>(max_nj, max_nc, 1, kBlock);
  hipLaunchKernelGGL(deflated_apply_kernel<T>, dim3(nsub), dim3(kBlock), lds, st, subs, cs, fac, Ec, v, w,
                     max_nj, max_nc);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kBlock) restrict_kernel(const SubDesc* __restrict__ subs,
                                                           const cplx<double>* __restrict__ v,
                                                           cplx<double>* __restrict__ t) {
  const SubDesc d = subs[blockIdx.x];
  restrict_to(d, v + d.off, t + d.coff, false);
}

hipError_t launch_restrict(const SubDesc* subs, int nsub, const cplx<double>* v, cplx<double>* t,
                           hipStream_t st) {
  hipLaunchKernelGGL(restrict_kernel, dim3(nsub), dim3(kBlock), 0, st, subs, v, t);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kBlock) prolong_kernel(const SubDesc* __restrict__ subs,
                                                          const cplx<double>* __restrict__ y,
                                                          cplx<double>* __restrict__ v) {
  const SubDesc d = subs[blockIdx.x];
  prolong_to(d, y + d.coff, v + d.off);
}

hipError_t launch_prolong(const SubDesc* subs, int nsub, const cplx<double>* y, cplx<double>* v,
                          hipStream_t st) {
  hipLaunchKernelGGL(prolong_kernel, dim3(nsub), dim3(kBlock), 0, st, subs, y, v);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kBlock) coarse_solve_kernel(const SubDesc* __restrict__ subs,
                                                               const cplx<double>* __restrict__ fac,
                                                               const cplx<double>* __restrict__ Ec,
                                                               const cplx<double>* __restrict__ t,
                                                               cplx<double>* __restrict__ y, int max_nc) {
  extern __shared__ __align__(16) unsigned char smem[];
  const SubDesc d = subs[blockIdx.x];
  cplx<double>* ct = (cplx<double>*)smem;
  cplx<double>* ca = ct + max_nc;
  cplx<double>* lc = ca + max_nc;
  cplx<double>* scr = lc + lower_entries(max_nc);
  const int nc = d.mx * d.my;
  for (int c = threadIdx.x; c < d.ncp; c += blockDim.x) ct[c] = c < nc ? t[d.coff + c] : czero<double>();
  stage_lower(d, Ec, lc);
  __syncthreads();
  const int kind = coarse_kind(d.defl, d.mx);
  if (kind == kCoarseNarrow) coarse_solve<kBlock, kCoarseNarrow>(d, fac, lc, ct, ca, scr, []() {});
  else if (kind == kCoarseChain) coarse_solve<kBlock, kCoarseChain>(d, fac, lc, ct, ca, scr, []() {});
  else coarse_solve<kBlock, kCoarseGeneral>(d, fac, lc, ct, ca, scr, []() {});
  for (int c = threadIdx.x; c < nc; c += blockDim.x) y[d.coff + c] = ca[c];
}

hipError_t launch_coarse_solve(const SubDesc* subs, int nsub, const cplx<double>* fac, const cplx<double>* Ec,
                               const cplx<double>* t, cplx<double>* y, int max_nc, hipStream_t st) {
  const size_t lds = (2 * (size_t)max_nc + lower_entries(max_nc) + detail::kChainScratch) * sizeof(cplx<double>);
  hipLaunchKernelGGL(coarse_solve_kernel, dim3(nsub), dim3(kBlock), lds, st, subs, fac, Ec, t, y, max_nc);
  return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(kBlock) gather_kernel(const SubDesc* __restrict__ subs, Consts cs,
                                                         const cplx<double>* __restrict__ r,
                                                         cplx<T>* __restrict__ f, long long nfine,
                                                         long long ndof) {
  const SubDesc d = subs[blockIdx.x];
  const int rhs = blockIdx.y, nj = d.nx * d.ny, ldg = cs.n - 1;
  for (int n = threadIdx.x; n < nj; n += blockDim.x) {
    const int lj = n / d.nx, li = n - lj * d.nx;
    f[rhs * nfine + d.off + n] =
        ccast<T>(r[rhs * ndof + (long long)(d.j0 + lj - 1) * ldg + (d.i0 + li - 1)]);
  }
}

template <typename T>
hipError_t launch_gather(const SubDesc* subs, int nsub, Consts cs, const cplx<double>* r, cplx<T>* f,
                         long long nfine, long long ndof, int nrhs, hipStream_t st) {
  hipLaunchKernelGGL(gather_kernel<T>, dim3(nsub, nrhs), dim3(kBlock), 0, st, subs, cs, r, f, nfine, ndof);
  return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(kBlock) scatter_kernel(const SubDesc* __restrict__ subs, Consts cs,
                                                          const cplx<T>* __restrict__ u,
                                                          cplx<double>* __restrict__ z, long long nfine,
                                                          long long ndof) {
  const SubDesc d = subs[blockIdx.x];
  const int rhs = blockIdx.y, ldg = cs.n - 1;
  const int ow = d.oi1 - d.oi0 + 1, oh = d.oj1 - d.oj0 + 1;
  for (int n = threadIdx.x; n < ow * oh; n += blockDim.x) {
    const int gj = d.oj0 + n / ow, gi = d.oi0 + n % ow;
    const int li = gi - d.i0, lj = gj - d.j0;
    z[rhs * ndof + (long long)(gj - 1) * ldg + (gi - 1)] = ccast<double>(u[rhs * nfine + d.off + lj * d.nx + li]);
  }
}

template <typename T>
hipError_t launch_scatter(const SubDesc* subs, int nsub, Consts cs, const cplx<T>* u, cplx<double>* z,
                          long long nfine, long long ndof, int nrhs, hipStream_t st) {
  hipLaunchKernelGGL(scatter_kernel<T>, dim3(nsub, nrhs), dim3(kBlock), 0, st, subs, cs, u, z, nfine, ndof);
  return hipGetLastError();
}

template <typename T>
hipError_t configure_inner(int max_nj, int max_nc, int maxit) {
  int dev = 0, maxlds = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&maxlds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  // A kernel whose LDS at these sizes exceeds the device limit is left unconfigured: set-up
  // has already rejected the handle unless it never launches that kernel (exact local solves
  // do not run the subdomain GMRES), and a launch of it is refused by the runtime.
  auto set = [&](const void* fn, size_t lds) {
    if (e == hipSuccess && lds > 65536 && lds <= (size_t)maxlds)
      e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  };
  for (int kind = kCoarseNarrow; kind <= kCoarseGeneral; ++kind) {
    set((const void*)inner_kernel<T, kInnerThreads>(kind), lds_bytes<T>(max_nj, max_nc, maxit, kInnerThreads));
    set((const void*)inner_kernel<T, 256>(kind), lds_bytes<T>(max_nj, max_nc, maxit, 256));
  }
  set((const void*)deflated_apply_kernel<T>, lds_bytes<T>(max_nj, max_nc, 1, kBlock));
  set((const void*)local_apply_kernel<T>,
      align16(kClasses * kStencilPts * sizeof(cplx<T>)) + (size_t)max_nj * sizeof(cplx<T>));
  set((const void*)coarse_solve_kernel, (2 * (size_t)max_nc + lower_entries(max_nc) + detail::kChainScratch) * sizeof(cplx<double>));
  return e;
}

#define DDH_INSTANTIATE(T)                                                                                   \
  template hipError_t launch_inner_solve<T>(const InnerArgs<T>&, hipStream_t);                                \
  template hipError_t configure_inner<T>(int, int, int);                                                     \
  template size_t inner_lds_bytes<T>(int, int, int);                                                          \
  template hipError_t launch_local_apply<T>(const SubDesc*, int, Consts, int, const cplx<T>*, cplx<T>*, int,  \
                                            hipStream_t);                                                     \
  template hipError_t launch_deflated_apply<T>(const SubDesc*, int, Consts, int, const cplx<double>*,         \
                                               const cplx<double>*, const cplx<T>*, cplx<T>*, int, int,       \
                                               hipStream_t);                                                  \
  template hipError_t launch_gather<T>(const SubDesc*, int, Consts, const cplx<double>*, cplx<T>*, long long, \
                                       long long, int, hipStream_t);                                          \
  template hipError_t launch_scatter<T>(const SubDesc*, int, Consts, const cplx<T>*, cplx<double>*, long long, \
                                        long long, int, hipStream_t);

DDH_INSTANTIATE(float)
DDH_INSTANTIATE(double)

}  // namespace ddh
