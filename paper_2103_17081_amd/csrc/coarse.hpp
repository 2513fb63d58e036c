// Coarse deflation operator E = Z^T B Z (Sec. 2, eq. 4) for linear interpolation
// Z = Z^y kron Z^x (eq. 5), and its FP64 block factorisations.
//
// With coarse nodes ordered x fastest, E couples a coarse node only to its 3 x 3
// coarse neighbours, so E is block tridiagonal in the coarse rows: diagonal blocks
// D_i, sub-diagonal L_i (row i to row i-1), super-diagonal U_i (row i to row i+1),
// each an mx x mx tridiagonal matrix.  E is complex symmetric (B is), so U_i = L_{i+1}^T;
// the factorisation and the solve both take U_i from the stored L_{i+1}, which keeps the
// factored matrix exactly symmetric whatever the rounding of the assembly.
//
// Twisted block factorisation (elimination from both ends towards the middle row
// p = (my - 1) / 2), without block pivoting:
//   top,    i < p:  G_i = (D_i - L_i G_{i-1} U_{i-1})^{-1};
//   bottom, i > p:  G_i = (D_i - U_i G_{i+1} L_{i+1})^{-1};
//   middle:         G_p = (D_p - L_p G_{p-1} U_{p-1} - U_p G_{p+1} L_{p+1})^{-1}.
// Solve E y = t:
//   a_i = G_i (t_i - L_i a_{i-1}) for i < p  and  a_i = G_i (t_i - U_i a_{i+1}) for i > p,
//   both sweeps side by side;  y_p = G_p (t_p - L_p a_{p-1} - U_p a_{p+1});
//   y_i = a_i - G_i U_i y_{i+1} (i < p)  and  y_i = a_i - G_i L_i y_{i-1} (i > p), side by side.
// The couplings are tridiagonal, so applying them costs three products per unknown; keeping
// G_i U_i and G_i L_i as dense blocks of their own would double the stored bytes.  Each
// inverse is formed by Gauss-Jordan elimination with partial pivoting.
//
// Storage per subdomain at SubDesc::goff (complex<double>): G_0 .. G_{my-1}, each mx*mx with
// element (r, c) at c*mx + r, so that consecutive lanes, which own consecutive rows, read
// consecutive entries.  E itself is kept as nine coefficients per coarse node, offset
// index o = 3*(dy+1) + (dx+1) for the neighbour (cx+dx, cy+dy).
//
// The exact local solves factor the local matrices B_j the same way (block size nx, ny
// block rows), through the same set-up kernel.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace ddh {

constexpr int kMaxMx = 128;   // largest coarse block (mx) the kernels support

__host__ __device__ __forceinline__ long long coarse_factor_size(int mx, int my) {
  return (long long)my * mx * mx;
}

// Middle row of the twisted factorisation.
__host__ __device__ __forceinline__ int twist_row(int my) { return (my - 1) / 2; }

// Bezier deflation couples coarse nodes up to two rows apart, so its E is taken as
// block tridiagonal over pairs of coarse rows (block size bmx = 2 mx, bmy block rows; an
// odd last row is padded with an identity row).  Its factors: G_0..G_{bmy-1},
// H_0..H_{bmy-2}, then the dense lower couplings L_1..L_{bmy-1}, each bmx x bmx
// row-major.  The solve is a_I = G_I (t_I - L_I a_{I-1}), y_I = a_I - H_I y_{I+1}.
__host__ __device__ __forceinline__ long long coarse_factor_size_paired(int bmx, int bmy) {
  return (long long)(3 * bmy - 2) * bmx * bmx;
}

// Factor entries (complex<double>) one coarse solve of subdomain d reads, plus the
// staged lower couplings of E for linear deflation.
__host__ __device__ __forceinline__ long long coarse_solve_values(const SubDesc& d) {
  return d.defl == 0 ? coarse_factor_size(d.mx, d.my) + 3LL * d.mx * d.my
                     : coarse_factor_size_paired(d.bmx, d.bmy);
}

// Lanes per block row in the coarse solve: the largest power of two up to 16 with
// lanes * mx <= NT.
template <int NT>
__host__ __device__ __forceinline__ int coarse_group_lanes(int mx) {
  int l = 1;
  while (l < 16 && 2 * l * mx <= NT) l *= 2;
  return l;
}

// Copy the three lower couplings of every coarse node of E (neighbours (cx-1..cx+1,
// cy-1), offsets o = 0, 1, 2; 0 outside the coarse grid) into LDS: lc[3 c + e], and a zero after
// the last one (lower_entries in all).  Workgroup-cooperative; the caller synchronises before the
// first coarse_solve.
__host__ __device__ __forceinline__ constexpr size_t lower_entries(size_t nc) { return 3 * nc + 1; }
__device__ __forceinline__ void stage_lower(const SubDesc& d, const cplx<double>* __restrict__ Ec,
                                            cplx<double>* lc) {
  if (d.defl != 0) return;   // the paired (Bezier) solve keeps its couplings with the factors
  const int nc = d.mx * d.my;
  const cplx<double>* ec = Ec + d.coff * 9;
  for (int e = threadIdx.x; e < 3 * nc; e += blockDim.x) lc[e] = ec[(size_t)(e / 3) * 9 + e % 3];
  if (threadIdx.x == 0) lc[3 * nc] = czero<double>();
}

namespace detail {

// ---- twisted solve of E (linear deflation; layout above) ----------------------------
// a and y share the LDS array `a` (row i at a + i mx); t is used as scratch.
// lower(i, c, e): coupling of unknown c of row i to unknown c+e-1 of row i-1 (for E, the
// staged lc[3 (i mx + c) + e]); the upper coupling of unknown c of row i-1 to c+e-1 of
// row i is lower(i, c+e-1, 2-e).

// `v` if `keep`, else 0 (a select, not a branch).
__device__ __forceinline__ cplx<double> keep_c(bool keep, cplx<double> v) {
  return cplx<double>{keep ? v.re : 0.0, keep ? v.im : 0.0};
}

// The three couplings of unknown c of row i to row i + dir (dir -1 or +1), unknowns c-1, c,
// c+1; those outside the row are 0 and read at c.
template <typename Lower>
__device__ __forceinline__ void tw_couplings(int mx, Lower lower, int i, int c, int dir, cplx<double> k[3]) {
  const bool lo = c > 0, hi = c < mx - 1;
  if (dir < 0) {
    k[0] = keep_c(lo, lower(i, c, 0));
    k[1] = lower(i, c, 1);
    k[2] = keep_c(hi, lower(i, c, 2));
  } else {
    k[0] = keep_c(lo, lower(i + 1, lo ? c - 1 : c, 2));
    k[1] = lower(i + 1, c, 1);
    k[2] = keep_c(hi, lower(i + 1, hi ? c + 1 : c, 0));
  }
}

// v - (couplings of unknown c of row i to row i + dir) x, x that row's values.
template <typename Lower>
__device__ __forceinline__ cplx<double> tw_couple(int mx, Lower lower, int i, int c, int dir, cplx<double> v,
                                                  const cplx<double>* x) {
  cplx<double> k[3];
  tw_couplings(mx, lower, i, c, dir, k);
  const cplx<double> xm = x[c > 0 ? c - 1 : c], x0 = x[c], xp = x[c < mx - 1 ? c + 1 : c];
  v = v - k[1] * x0;
  v = v - k[0] * xm;
  return v - k[2] * xp;
}

// Orders this wave's LDS accesses before those after it (the LDS unit serves one wave's
// operations in order, so nothing has to be waited for).
__device__ __forceinline__ void wave_lds_order() { asm volatile("" ::: "memory"); }

// Sum of v over the lanes l, l + 64 / L, l + 2 * 64 / L, ... (L = 2, 4 or 8); all of them get it.
template <int L>
__device__ __forceinline__ double column_sum(double v) {
  if constexpr (L == 8) v += dpp_f64<kDppRowRor8>(v);
  if constexpr (L >= 4) v = fold16(v, v);
  return fold32(v, v);
}

// Value of the neighbouring row's lane (row - 1 / row + 1); the rows of a wave are its lanes
// modulo 64 / L: 16-lane rows of the wave for L = 4, the half wave for L = 2 (the lane past the
// end gets another column group's value, always multiplied by a coupling of 0).
constexpr int kDppRowShr1 = 0x111, kDppRowShl1 = 0x101, kDppWaveShr1 = 0x138, kDppWaveShl1 = 0x130;
template <int L>
__device__ __forceinline__ cplx<double> row_below(cplx<double> v) {
  constexpr int ctrl = L == 4 ? kDppRowShr1 : kDppWaveShr1;
  return cplx<double>{dpp_f64<ctrl>(v.re), dpp_f64<ctrl>(v.im)};
}
template <int L>
__device__ __forceinline__ cplx<double> row_above(cplx<double> v) {
  constexpr int ctrl = L == 4 ? kDppRowShl1 : kDppWaveShl1;
  return cplx<double>{dpp_f64<ctrl>(v.re), dpp_f64<ctrl>(v.im)};
}

// Entries allocated (and zeroed) after the last factor block, for the columns a lane of the chain
// reads past the end of a block.
constexpr int kFactorPad = 32 * 32;

// Entries of the LDS scratch of coarse_solve (one vector per half of the workgroup).
constexpr int kChainScratch = 2 * 32;

// The solve as a chain of waves, mx <= L Q and mx <= 64 / L.  The waves of a workgroup form two
// halves, one per sweep; each wave owns `per` consecutive block rows of its half's sweep and
// holds their G_i in registers from the forward to the backward pass (Slots blocks; further
// ones are fetched again when a slot is free), all loads issued before the first step.  A step
// is one wave's work: lane r + (64 / L) g owns row r and the columns g + q L, forms the coupled
// right-hand side with its neighbours' values (DPP), shares it through LDS with its own wave
// only, multiplies and sums over g with lane swaps.  Only handing the sweep to the next wave
// takes a workgroup barrier, instead of one or two for every block row.
//
// What bounds it: the dependent steps (my of them forward and backward, 0.2 us each: an LDS
// round trip, 4 Q FP64 FMAs, the lane swaps), no longer the latency of the factor loads.
template <int NT, int L, int Q, int Slots>
struct CoarseChain {
  static constexpr int kHalfWaves = NT / (2 * kWave);
  static constexpr int kBatch = 4;
  cplx<double> G[Slots][Q];
  int mx, my, p, half, pos, per, first, count, r, g;
  unsigned off;

  // block row of position s of this wave's half (top: 0 .. p, bottom: my - 1 .. p + 1)
  __device__ __forceinline__ int row_of(int s) const { return half ? my - 1 - s : s; }

  // Columns past the block read what follows it in the factor array (kFactorPad entries follow
  // the last block) and multiply zeros.
  __device__ __forceinline__ void load(cplx<double> (&dst)[Q], const cplx<double>* __restrict__ F, int s) {
    const cplx<double>* B = F + (size_t)(row_of(s) * mx * mx);   // uniform: scalar base, one lane offset
#pragma unroll
    for (int q = 0; q < Q; ++q) dst[q] = (B + q * L * mx)[off];
  }

  // Split the block rows over the waves and issue the loads of the first blocks.
  __device__ __forceinline__ void start(int mx_, int my_, const cplx<double>* __restrict__ F) {
    mx = mx_;
    my = my_;
    p = twist_row(my);
    const int tid = fresh_tid(), lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    half = wave / kHalfWaves;
    // the halves' active waves sit on different SIMDs (waves w and w + 4 share one)
    pos = half ? (wave + kHalfWaves / 2) % kHalfWaves : wave;
    r = min(lane % (kWave / L), mx - 1);   // spare lanes repeat the last row
    g = lane / (kWave / L);
    off = (unsigned)(g * mx + r);
    const int longest = max(p + 1, my - 1 - p);
    per = max((longest + kHalfWaves - 1) / kHalfWaves, min(longest, Slots));
    const int n = half ? my - 1 - p : p + 1;
    first = pos * per;
    count = max(0, min(per, n - first));
#pragma unroll
    for (int k = 0; k < Slots; ++k)
      if (k < count) load(G[k], F, first + k);
  }

  // What a step reads besides the factor block: the couplings of unknown r of block row i to row
  // i + dir and entry r of row i of `rhs`.  Read one step ahead: it does not depend on the chain.
  struct Inputs {
    cplx<double> k[3], rhs;
  };
  template <typename Lower>
  __device__ __forceinline__ Inputs fetch(Lower lower, int i, int dir, const cplx<double>* rhs) const {
    Inputs in;
    if constexpr (std::is_pointer_v<Lower>) {
      // lower couplings of row i, or those of row i + 1 transposed; the ones that leave the row are
      // stored zeros (the last entry is stage_lower's padding)
      const cplx<double>* e = lower + 3 * (min(i + (dir > 0 ? 1 : 0), my - 1) * mx + r);
      in.k[0] = e[dir > 0 ? -1 : 0];
      in.k[1] = e[1];
      in.k[2] = e[dir > 0 ? 3 : 2];
    } else {
      tw_couplings(mx, lower, dir > 0 ? min(i, my - 2) : i, r, dir, in.k);
    }
    in.rhs = rhs[i * mx + r];
    return in;
  }

  // Couplings of the step's row to the neighbouring block row's values.
  __device__ __forceinline__ cplx<double> coupled(const Inputs& in, cplx<double> prev) const {
    const cplx<double> xm = row_below<L>(prev), xp = row_above<L>(prev);
    cplx<double> v = in.k[1] * prev;
    v = cfma(in.k[0], xm, v);
    return cfma(in.k[2], xp, v);
  }

  // Row r of B x, x entry r held as v; `next` is filled while the product runs.
  template <typename Next>
  __device__ __forceinline__ cplx<double> product(const cplx<double> (&B)[Q], cplx<double> v, cplx<double>* xb,
                                                  Next next) const {
    const int lane = threadIdx.x % kWave;
    wave_lds_order();
    if (g == 0) xb[lane] = keep_c(lane < mx, v);   // columns past the row multiply zeros
    wave_lds_order();
    // x in batches, one ahead of the products: few values live at a time
    cplx<double> acc[2] = {czero<double>(), czero<double>()}, x[2][kBatch];
    auto read = [&](int b) {
#pragma unroll
      for (int q = b * kBatch; q < (b + 1) * kBatch && q < Q; ++q) x[b % 2][q - b * kBatch] = xb[g + q * L];
    };
    read(0);
#pragma unroll
    for (int b = 0; b * kBatch < Q; ++b) {
      if ((b + 1) * kBatch < Q) read(b + 1);
      if ((b + 1) * kBatch >= Q) next();
      wave_lds_order();
#pragma unroll
      for (int q = b * kBatch; q < (b + 1) * kBatch && q < Q; ++q)
        acc[q % 2] = cfma(B[q], x[b % 2][q - b * kBatch], acc[q % 2]);
    }
    const cplx<double> acc0 = acc[0] + acc[1];
    return cplx<double>{column_sum<L>(acc0.re), column_sum<L>(acc0.im)};
  }

  // `lc`: the couplings staged by stage_lower, or a function lower(i, c, e) as above.
  template <typename Lower>
  __device__ __forceinline__ void solve(const cplx<double>* __restrict__ F, Lower lc, cplx<double>* t,
                                        cplx<double>* a, cplx<double>* scratch) {
    const bool writes = threadIdx.x % kWave < mx && g == 0;
    cplx<double>* xb = scratch + half * 32;
    const int fdir = half ? 1 : -1;
    const int rounds = (max(p + 1, my - 1 - p) + per - 1) / per;
    const int last = half ? first + count - 1 : min(first + count, p) - 1;   // last position but the middle row
    cplx<double> prev = czero<double>();   // entry r of the neighbouring block row (0 before the first)
    // forward: a_i = G_i (t_i - couplings to the row before it in the sweep)
    for (int w = 0; w < rounds; ++w) {
      if (w == pos && last >= first) {
        Inputs in = fetch(lc, row_of(first), fdir, t);
        if (first > 0) prev = a[row_of(first - 1) * mx + r];
        for (int u0 = 0; u0 < count; u0 += Slots) {
#pragma unroll
          for (int k = 0; k < Slots; ++k) {
            const int u = u0 + k, s = first + u;
            if (s <= last) {
              const cplx<double> v = in.rhs - coupled(in, prev);
              prev = product(G[k], v, xb, [&]() { in = fetch(lc, row_of(min(s + 1, last)), fdir, t); });
              if (writes) a[row_of(s) * mx + r] = prev;
              if (u + Slots < count) load(G[k], F, s + Slots);
            }
          }
        }
      }
      lds_barrier();
    }
    // the middle row, by the wave that owns it
    if (!half && count > 0 && first + count - 1 == p) {
      cplx<double> v = t[p * mx + r];
      auto lower = [lc, this](int i, int c, int e) {
        if constexpr (std::is_pointer_v<Lower>) return lc[3 * (i * mx + c) + e];
        else return lc(i, c, e);
      };
      if (p > 0) v = tw_couple(mx, lower, p, r, -1, v, a + (p - 1) * mx);
      if (p < my - 1) v = tw_couple(mx, lower, p, r, 1, v, a + (p + 1) * mx);
      const int km = (count - 1) % Slots;
      cplx<double> y = czero<double>();
#pragma unroll
      for (int k = 0; k < Slots; ++k)
        if (k == km) {
          y = product(G[k], v, xb, []() {});
          if (count - 1 >= Slots) load(G[k], F, p - Slots);
        }
      if (writes) a[p * mx + r] = y;
    }
    lds_barrier();
    // backward: y_i = a_i - G_i (couplings to the row after it in the sweep)
    for (int w = rounds - 1; w >= 0; --w) {
      if (w == pos && last >= first) {
        Inputs in = fetch(lc, row_of(last), -fdir, a);
        prev = a[row_of(last + 1) * mx + r];
        for (int u0 = (count - 1) / Slots * Slots; u0 >= 0; u0 -= Slots) {
#pragma unroll
          for (int k = Slots - 1; k >= 0; --k) {
            const int u = u0 + k, s = first + u;
            if (s <= last) {
              const cplx<double> ai = in.rhs, v = coupled(in, prev);
              prev = ai - product(G[k], v, xb, [&]() { in = fetch(lc, row_of(max(s - 1, first)), -fdir, a); });
              if (writes) a[row_of(s) * mx + r] = prev;
              if (u >= Slots) load(G[k], F, s - Slots);
            }
          }
        }
      }
      lds_barrier();
    }
  }
};

// The same steps for wider block rows, one step of both sweeps at a time for the whole
// workgroup (half 0 the top sweep and the middle row, half 1 the bottom sweep):
//   s < nf = my - 1 - p:  a_s (top, if s < p) and a_{my-1-s} (bottom);
//   s = nf:               y_p;
//   s > nf:               y_{p-1-(s-nf-1)} (top) and y_{p+1+(s-nf-1)} (bottom).
// A step forms the coupled right-hand side, then the block product.

// Block row of half h at step s, or -1.
__device__ __forceinline__ int tw_step_row(int h, int s, int p, int my) {
  const int nf = my - 1 - p;
  if (s < nf) return h == 0 ? (s < p ? s : -1) : my - 1 - s;
  if (s == nf) return h == 0 ? p : -1;
  const int i = h == 0 ? p - (s - nf) : p + (s - nf);
  return i >= 0 && i < my ? i : -1;
}

// Coupled right-hand side of unknown c of row i at step s.
template <typename Lower>
__device__ __forceinline__ cplx<double> tw_step_rhs(int mx, int my, int p, Lower lower, int h, int s, int i, int c,
                                                    const cplx<double>* t, const cplx<double>* a) {
  const int nf = my - 1 - p;
  if (s <= nf) {
    cplx<double> v = t[i * mx + c];
    if (i <= p && i > 0) v = tw_couple(mx, lower, i, c, -1, v, a + (i - 1) * mx);
    if (i >= p && i < my - 1) v = tw_couple(mx, lower, i, c, 1, v, a + (i + 1) * mx);
    return v;
  }
  const int dir = h == 0 ? 1 : -1;
  return czero<double>() - tw_couple(mx, lower, i, c, dir, czero<double>(), a + (i + dir) * mx);
}

// The lanes of a wave own 64 / L consecutive rows, so a lane group's load of a column is contiguous; group l
// owns columns l + q L, q < Q (mx <= L Q, rows Half / L >= mx).  The next step's factor block is loaded into the
// registers that a step's product has just read.  With `own` (64 entries per wave; mx <= 64) every
// wave forms the coupled right-hand side for itself, a lane per unknown, which leaves one barrier per step;
// without, the half forms it in t, with a barrier of its own.
// Bound by latency with few subdomains (a step is the wait for its factors, the sum over the lane groups and
// the barrier), by the factor bytes with many.  Exact solves (Own), us per application, lanes of a row next to each other
// (four columns at a stride of one column: up to 1.5 times the time where mx is a multiple of 8), two barriers and the loads
// of a step at its start -> this: 4 subdomains of 49 nodes 126 -> 81, 64 of 48 nodes 138 -> 76, 64 of 61
// nodes 176 -> 130, 256 of 45 nodes 121 -> 112.  Two blocks ahead: the same above 40 nodes, 4 us more below.
template <int L, int Q, int Half, bool Own, typename Lower>
__device__ __forceinline__ void twisted_solve_ring(int mx, int my, const cplx<double>* __restrict__ F, Lower lower,
                                                   cplx<double>* t, cplx<double>* a, cplx<double>* own = nullptr) {
  constexpr int kRows = kWave / L;
  const int mm = mx * mx, p = twist_row(my), nf = my - 1 - p, nsteps = 2 * nf + 1;
  const int h = threadIdx.x / Half, ht = threadIdx.x % Half, lane = threadIdx.x % kWave;
  const int r = ht / kWave * kRows + lane % kRows, l = lane / kRows;
  const bool active = r < mx;
  // Columns past the row read entry 0 of the block and multiply it by 0, so every step reads its
  // operands without branches (adding 0 * x leaves the sum unchanged).
  int col[Q], eoff[Q];
  bool ok[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    ok[q] = active && l + q * L < mx;
    col[q] = Own || ok[q] ? l + q * L : 0;
    eoff[q] = ok[q] ? col[q] * mx + r : 0;
  }
  if (Own) own += threadIdx.x / kWave * kWave;
  cplx<double> G[Q];
  auto load = [&](int s) {
    const cplx<double>* B = F + (size_t)max(tw_step_row(h, s, p, my), 0) * mm;
#pragma unroll
    for (int q = 0; q < Q; ++q) G[q] = B[eoff[q]];
  };
  load(0);
  for (int s = 0; s < nsteps; ++s) {
    const int i = tw_step_row(h, s, p, my);
    const cplx<double>* x = t + i * mx;
    if constexpr (Own) {
      wave_lds_order();
      if (i >= 0) own[lane] = lane < mx ? tw_step_rhs(mx, my, p, lower, h, s, i, lane, t, a) : czero<double>();
      wave_lds_order();
      x = own;
    } else {
      if (i >= 0 && ht < mx) t[i * mx + ht] = tw_step_rhs(mx, my, p, lower, h, s, i, ht, t, a);
      lds_barrier();
    }
    cplx<double> acc = czero<double>();
    if (i >= 0) {
#pragma unroll
      for (int q = 0; q < Q; ++q) acc = cfma(G[q], Own ? x[col[q]] : keep_c(ok[q], x[col[q]]), acc);
    }
    load(s + 1);
    acc.re = column_sum<L>(acc.re);
    acc.im = column_sum<L>(acc.im);
    if (i >= 0 && active && l == 0) a[i * mx + r] = s <= nf ? acc : a[i * mx + r] - acc;
    lds_barrier();
  }
}

// Same steps for any mx <= kMaxMx: factor entries read as they are used, shuffle
// reductions over groups of L = coarse_group_lanes<Half>(mx) lanes.
template <int Half, typename Lower>
__device__ __forceinline__ void twisted_solve_plain(int mx, int my, const cplx<double>* __restrict__ F, Lower lower,
                                                    cplx<double>* t, cplx<double>* a) {
  const int mm = mx * mx, p = twist_row(my), nf = my - 1 - p, nsteps = 2 * nf + 1;
  const int L = coarse_group_lanes<Half>(mx);
  const int h = threadIdx.x / Half, ht = threadIdx.x % Half;
  const int r = ht / L, l = ht % L;
  const bool active = r < mx;
  auto gsum = [&](cplx<double> v) {
    for (int o = L >> 1; o > 0; o >>= 1) {
      v.re += __shfl_xor(v.re, o, kWave);
      v.im += __shfl_xor(v.im, o, kWave);
    }
    return v;
  };
  for (int s = 0; s < nsteps; ++s) {
    const int i = tw_step_row(h, s, p, my);
    if (i >= 0 && ht < mx) t[i * mx + ht] = tw_step_rhs(mx, my, p, lower, h, s, i, ht, t, a);
    lds_barrier();
    cplx<double> acc = czero<double>();
    if (i >= 0 && active)
      for (int c = l; c < mx; c += L) acc = cfma(F[(size_t)i * mm + c * mx + r], t[i * mx + c], acc);
    acc = gsum(acc);
    if (i >= 0 && active && l == 0) a[i * mx + r] = s <= nf ? acc : a[i * mx + r] - acc;
    lds_barrier();
  }
}

// Paired-row (Bezier) block solve with dense lower couplings; shuffle reductions over
// groups of L lanes, one LDS barrier per block product.
template <int NT>
__device__ __forceinline__ void coarse_solve_paired(const SubDesc& d, const cplx<double>* __restrict__ F,
                                                    cplx<double>* t, cplx<double>* a) {
  const int bm = d.bmx, bn = d.bmy, mm = bm * bm;
  const int L = coarse_group_lanes<NT>(bm);
  const int r = threadIdx.x / L, l = threadIdx.x % L;
  const bool active = r < bm;
  auto gsum = [&](cplx<double> v) {
    for (int o = L >> 1; o > 0; o >>= 1) {
      v.re += __shfl_xor(v.re, o, kWave);
      v.im += __shfl_xor(v.im, o, kWave);
    }
    return v;
  };
  for (int I = 0; I < bn; ++I) {
    if (I > 0) {
      const cplx<double>* Lb = F + (size_t)(2 * bn - 2 + I) * mm;
      cplx<double> acc = czero<double>();
      if (active)
        for (int c = l; c < bm; c += L) acc = cfma(Lb[r * bm + c], a[(I - 1) * bm + c], acc);
      acc = gsum(acc);
      if (active && l == 0) t[I * bm + r] = t[I * bm + r] - acc;
      lds_barrier();
    }
    const cplx<double>* G = F + (size_t)I * mm;
    cplx<double> acc = czero<double>();
    if (active)
      for (int c = l; c < bm; c += L) acc = cfma(G[r * bm + c], t[I * bm + c], acc);
    acc = gsum(acc);
    if (active && l == 0) a[I * bm + r] = acc;
    lds_barrier();
  }
  for (int I = bn - 2; I >= 0; --I) {
    const cplx<double>* H = F + (size_t)(bn + I) * mm;
    cplx<double> acc = czero<double>();
    if (active)
      for (int c = l; c < bm; c += L) acc = cfma(H[r * bm + c], a[(I + 1) * bm + c], acc);
    acc = gsum(acc);
    if (active && l == 0) a[I * bm + r] = a[I * bm + r] - acc;
    lds_barrier();
  }
}

}  // namespace detail

// Form of the coarse solve, compiled into kernels of their own (a kernel's registers are those of
// its largest form): the wave chain with 4 lanes per row (linear deflation, mx <= 16), with 2 lanes of
// 13 columns (mx <= 26), or the step-by-step forms and the paired rows of Bezier deflation.  The chain of 13 columns
// takes all 256 registers of a 512-thread kernel.  One tile past 53 nodes moves every subdomain of its
// handle to the step-by-step form; an application of 16 complex64 solves then takes (us, twice the factor bytes and dependent
// stored products -> two barriers -> this) 1097 -> 1029 -> 935 at 54 nodes, 1472 -> 1365 -> 1244 at 61, against 682 at 53.
enum CoarseKind { kCoarseNarrow = 0, kCoarseChain = 1, kCoarseGeneral = 2 };
constexpr int kNarrowMx = 16, kChainMx = 26;

// The form that covers every subdomain of a set with these block widths.
__host__ __device__ __forceinline__ int coarse_kind(int defl, int max_mx) {
  return defl != 0 || max_mx > kChainMx ? kCoarseGeneral : (max_mx <= kNarrowMx ? kCoarseNarrow : kCoarseChain);
}

// y = E^{-1} t for one subdomain, workgroup-cooperative (NT threads).  `t` and `a`
// are d.ncp-entry LDS arrays (must not alias; entries from mx * my on are zero
// padding); the result overwrites `a` and `t` is used as scratch (its content is
// lost); `lc` holds the lower couplings staged by stage_lower (linear deflation), `scratch`
// kChainScratch LDS entries.  `fac` is the handle's factor base (the subdomain offset is applied
// here).  `before` forms the right-hand side in `t` (ending in a workgroup barrier); it runs with
// the first factor blocks already on their way.
template <int NT, int Kind, typename Before>
__device__ __forceinline__ void coarse_solve(const SubDesc& d, const cplx<double>* __restrict__ fac,
                                             const cplx<double>* lc, cplx<double>* t, cplx<double>* a,
                                             cplx<double>* scratch, Before before) {
  const cplx<double>* __restrict__ F = fac + d.goff;
  if constexpr (Kind == kCoarseNarrow) {
    detail::CoarseChain<NT, 4, 4, 6> ch;
    ch.start(d.mx, d.my, F);
    before();
    ch.solve(F, lc, t, a, scratch);
  } else if constexpr (Kind == kCoarseChain) {
    detail::CoarseChain<NT, 2, 13, 3> ch;
    ch.start(d.mx, d.my, F);
    before();
    ch.solve(F, lc, t, a, scratch);
  } else {
    before();
    if (d.defl != 0) {
      detail::coarse_solve_paired<NT>(d, F, t, a);
      return;
    }
    auto lower = [lc, mx = d.mx](int i, int c, int e) { return lc[3 * (i * mx + c) + e]; };
    if (d.mx <= 32) {
      if constexpr (NT >= 512) detail::twisted_solve_ring<8, 4, NT / 2, false>(d.mx, d.my, F, lower, t, a);
      else detail::twisted_solve_ring<4, 8, NT / 2, false>(d.mx, d.my, F, lower, t, a);
    } else {
      detail::twisted_solve_plain<NT / 2>(d.mx, d.my, F, lower, t, a);
    }
  }
}

}  // namespace ddh
