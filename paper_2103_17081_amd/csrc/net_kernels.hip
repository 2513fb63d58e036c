// Kernels of the learned initial guess (network layout and scaling in net.hpp).
//
// 3x3 layers are implicit GEMMs on v_mfma_f32_16x16x32_bf16: a workgroup stages a
// band of image rows (plus a one-pixel halo) of the layer input in LDS, applying the
// layer's input transform on the way (2x2 average pooling, or nearest upsampling of
// one operand concatenated with a skip operand), and each wave multiplies 16-pixel
// fragments of the staged band by pre-arranged weight fragments.  The data gradient
// of a layer is the same product with the weights flipped in space and transposed in
// channels; the weight gradient reduces im2col(input)^T dz over the pixels of bands of rows,
// one partial per workgroup, summed in a second kernel in a fixed order.
//
// MFMA operand layout (16x16x32): lane l supplies row l % 16 of A and column l % 16
// of B over the same 8 reduction indices (8 (l / 16) + e within the 32-wide step);
// lane l receives rows 4 (l / 16) + i, i < 4, of column l % 16 of the product.
#include <algorithm>

#include "net.hpp"
#include "stencil.hpp"

namespace ddh {

namespace {

__device__ __forceinline__ bf16x8 zero8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (bf16)0.0f;
  return z;
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 8 consecutive input channels (from ch) of layer-input pixel (y, x) of tile b.
__device__ __forceinline__ bf16x8 load_input(const ConvArgs& a, int b, int y, int x, int ch) {
  const int H = a.H, W = a.W;
  if (a.mode == kPlain) return *(const bf16x8*)(a.x0 + (((size_t)b * H + y) * W + x) * a.cinp + ch);
  if (a.mode == kInput) {
    const f32x4 v = *(const f32x4*)(a.xf + (((size_t)b * H + y) * W + x) * kNetIn);
    bf16x8 o = zero8();
#pragma unroll
    for (int i = 0; i < kNetIn; ++i) o[i] = (bf16)v[i];
    return o;
  }
  if (a.mode == kPool) {
    const int W2 = 2 * W;
    const bf16* base = a.x0 + (((size_t)b * 2 * H + 2 * y) * W2 + 2 * x) * a.cinp + ch;
    const bf16x8 v00 = *(const bf16x8*)base;
    const bf16x8 v01 = *(const bf16x8*)(base + a.cinp);
    const bf16x8 v10 = *(const bf16x8*)(base + (size_t)W2 * a.cinp);
    const bf16x8 v11 = *(const bf16x8*)(base + (size_t)W2 * a.cinp + a.cinp);
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      o[i] = (bf16)(0.25f * (((float)v00[i] + (float)v01[i]) + ((float)v10[i] + (float)v11[i])));
    return o;
  }
  if (ch < a.c1) {
    const int Hl = H >> 1, Wl = W >> 1;
    return *(const bf16x8*)(a.x0 + (((size_t)b * Hl + (y >> 1)) * Wl + (x >> 1)) * a.c1 + ch);
  }
  const int cs = a.cinp - a.c1;
  return *(const bf16x8*)(a.x1 + (((size_t)b * H + y) * W + x) * cs + (ch - a.c1));
}

// 16 bytes at a 32-bit byte offset from a uniform base.
template <typename V>
__device__ __forceinline__ V load_at(const void* base, int bytes) {
  return *(const V*)((const char*)base + (unsigned)bytes);
}

// 2^lcg groups of 8 channels of rows y0-1 .. y0+rows of a tile into LDS, columns 0 .. W-1, from channel c0
// (pixel stride ps, one pixel of halo on the left). The pixels of a band follow each other in memory, so a unit's
// place is its number: the address takes a shift, and pixel p of the band goes to LDS pixel
// p + 2 (p / W) + 1. Each thread issues its loads before it combines and stores any. Rows
// outside the tile are read at its first or last pixel and stored as zeros.
template <int MODE>
__device__ __forceinline__ void stage_rows(const ConvArgs& a, const void* src, int lcg, int y0, int rows, int ps,
                                           bf16* lds) {
  constexpr int kBatch = MODE == kPool ? 4 : 8, kLoads = MODE == kPool ? 4 : 1, nt = kNetThreads;
  const int n = (rows + 2) << a.lw << lcg, first = (y0 - 1) << a.lw, npix = a.H << a.lw;
  for (int u0 = 0; u0 < n; u0 += nt * kBatch) {
    bf16x8 v[kBatch][kLoads];
    f32x4 f[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      if (u0 + q * nt < n) {
        const int e = u0 + q * nt + threadIdx.x, g = e & ((1 << lcg) - 1);
        const int p = min(max(first + (e >> lcg), 0), npix - 1);
        if (MODE == kInput) {
          f[q] = load_at<f32x4>(src, p * 16);
        } else if (MODE == kPool) {
          const int at = (((4 * p - 2 * (p & (a.W - 1))) << lcg) + g) * 16;
          const int right = 16 << lcg, down = right << (a.lw + 1);
          v[q][0] = load_at<bf16x8>(src, at);
          v[q][kLoads > 1 ? 1 : 0] = load_at<bf16x8>(src, at + right);
          v[q][kLoads > 2 ? 2 : 0] = load_at<bf16x8>(src, at + down);
          v[q][kLoads > 3 ? 3 : 0] = load_at<bf16x8>(src, at + down + right);
        } else {
          v[q][0] = load_at<bf16x8>(src, ((p << lcg) + g) * 16);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      if (u0 + q * nt < n) {
        const int e = u0 + q * nt + threadIdx.x, g = e & ((1 << lcg) - 1), p = e >> lcg;
        bf16x8 o = zero8();
        if (MODE == kInput) {
#pragma unroll
          for (int i = 0; i < kNetIn; ++i) o[i] = (bf16)f[q][i];
        } else if (MODE == kPool) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            o[i] = (bf16)(0.25f * (((float)v[q][0][i] + (float)v[q][kLoads > 1 ? 1 : 0][i]) +
                                   ((float)v[q][kLoads > 2 ? 2 : 0][i] + (float)v[q][kLoads > 3 ? 3 : 0][i])));
        } else {
          o = v[q][0];
        }
        if ((unsigned)(first + p) >= (unsigned)npix) o = zero8();
        if (e < n) *(bf16x8*)(lds + (p + 2 * (p >> a.lw) + 1) * ps + g * 8) = o;
      }
    }
  }
}

// The same from a tile of half the resolution: each pixel is read once and stored to the up to four
// that it covers.
__device__ __forceinline__ void stage_upsampled(const ConvArgs& a, const void* src, int lcg, int y0, int rows, int ps,
                                                bf16* lds) {
  constexpr int kBatch = 4, nt = kNetThreads;
  const int lwc = a.lw - 1, npix = (a.H >> 1) << lwc;
  const int top = (y0 - 1) >> 1, first = top * (1 << lwc);   // y0 = 0: row -1
  const int n = (((y0 + rows) >> 1) - top + 1) << lwc << lcg;
  for (int u0 = 0; u0 < n; u0 += nt * kBatch) {
    bf16x8 v[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      if (u0 + q * nt < n) {
        const int e = u0 + q * nt + threadIdx.x, g = e & ((1 << lcg) - 1);
        const int p = min(max(first + (e >> lcg), 0), npix - 1);
        v[q] = load_at<bf16x8>(src, ((p << lcg) + g) * 16);
      }
    }
#pragma unroll
    for (int q = 0; q < kBatch; ++q) {
      if (u0 + q * nt < n) {
        const int e = u0 + q * nt + threadIdx.x, g = e & ((1 << lcg) - 1), p = e >> lcg;
        bf16x8 o = v[q];
        if ((unsigned)(first + p) >= (unsigned)npix) o = zero8();
        const int x = p & ((1 << lwc) - 1), r = 2 * (top + (p >> lwc)) - (y0 - 1);   // band row of the upper two
        bf16* d = lds + (r * (a.W + 2) + 2 * x + 1) * ps + g * 8;
        if (e < n && r >= 0) {
          *(bf16x8*)d = o;
          *(bf16x8*)(d + ps) = o;
        }
        if (e < n && r + 1 < rows + 2) {
          *(bf16x8*)(d + (a.W + 2) * ps) = o;
          *(bf16x8*)(d + (a.W + 3) * ps) = o;
        }
      }
    }
  }
}

// Rows y0-1 .. y0+rows of the layer input, columns -1 .. W, into LDS (pixel stride cinp + 8 channels).
__device__ __forceinline__ void stage_input(const ConvArgs& a, int b, int y0, int rows, bf16* lds) {
  const int ps = a.cinp + 8, lcg = a.lc - 3;
  const size_t pix = (size_t)b * a.H * a.W;
  for (int u = threadIdx.x; u < (rows + 2) << (lcg + 1); u += kNetThreads) {
    const int g = u & ((1 << lcg) - 1), e = u >> lcg;
    *(bf16x8*)(lds + ((e >> 1) * (a.W + 2) + (e & 1) * (a.W + 1)) * ps + g * 8) = zero8();
  }
  switch (a.mode) {
    case kPlain: stage_rows<kPlain>(a, a.x0 + pix * a.cinp, lcg, y0, rows, ps, lds); break;
    case kPool: stage_rows<kPool>(a, a.x0 + 4 * pix * a.cinp, lcg, y0, rows, ps, lds); break;
    case kInput: stage_rows<kInput>(a, a.xf + pix * kNetIn, lcg, y0, rows, ps, lds); break;
    default:   // both operands have half of the channels
      stage_upsampled(a, a.x0 + (pix >> 2) * a.c1, lcg - 1, y0, rows, ps, lds);
      stage_rows<kPlain>(a, a.x1 + pix * a.c1, lcg - 1, y0, rows, ps, lds + a.c1);
  }
}

}  // namespace

// LDS of one workgroup of a 3x3 product with MF fragments per wave: the staged band.
static size_t conv_lds_bytes(int H, int W, int cinp, int mf) {
  const int np = std::min(64 * mf, H * W);
  return (size_t)((np + W - 1) / W + 2) * (W + 2) * (cinp + 8) * sizeof(bf16);
}

// Fragments per wave. More of them read fewer halo rows and weights; fewer give a small
// batch more workgroups, each with less to stage before its first product. Two workgroups per compute
// unit are enough (against four: 256 tiles of 64 x 64 108 and 112 us, 4 of 128 x 128 43 and
// 49, one and 8 of 64 x 64 equal), and more than 80 KB of LDS would leave one.
static int conv_mf(int H, int W, int cinp, int nb, int batch) {
  int mf = nb >= 8 ? 2 : 4;
  while (mf > 1 && ((long long)batch * ((H * W + 64 * mf - 1) / (64 * mf)) < 512 ||
                    conv_lds_bytes(H, W, cinp, mf) > 80 * 1024))
    mf >>= 1;
  return mf;
}

// out[p][co] = bias[co] + sum_{tap, ci} in[p + off(tap)][ci] W[tap][ci][co]   (+ relu)
// Grid: (ceil(H W / (64 MF)), batch); 256 threads; wave w owns fragments w + 4 f.
//
// The weight fragments go from L2 straight to registers, kConvSteps steps ahead, the first
// before the band is staged: every wave needs all of them once, so LDS would only add a
// copy, a wait and up to 72 KB. Bound by vector instructions (staging, addresses, rounding) and
// the staging's latency; products are issued at 5 to 16% of the bf16 peak.
// Forward pass at widths 16/32/64/64 with weights in LDS and the head, input rounding and
// output copy in launches of their own: 217 us for 256 tiles of 64 x 64 and 113 for one, now 108 and 33.
//
// With a.y the 1x1 head follows in the same lanes, on the activations as rounded to bfloat16:
// y[p] = out[p] W8 + b8, and out itself is not stored.
template <int NB, int MF>
__global__ void __launch_bounds__(kNetThreads) conv3x3_kernel(ConvArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  bf16* lds = (bf16*)smem;
  const int b = blockIdx.y;
  const int W = a.W, npix = a.H * W;
  const int p0 = blockIdx.x * (64 * MF);
  const int np = min(64 * MF, npix - p0);
  const int y0 = p0 >> a.lw, rows = ((p0 + np - 1) >> a.lw) - y0 + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lg = lane >> 4;
  bf16x8 wv[kConvSteps][NB];
#pragma unroll
  for (int q = 0; q < kConvSteps; ++q)
#pragma unroll
    for (int n = 0; n < NB; ++n) wv[q][n] = load_at<bf16x8>(a.wf + (q * NB + n) * 64, lane * 16);
  stage_input(a, b, y0, rows, lds);
  __syncthreads();
  const int ps = a.cinp + 8, W2 = W + 2, steps = a.ksteps;
  f32x4 acc[MF][NB];
  const bf16* at[MF];
#pragma unroll
  for (int f = 0; f < MF; ++f) {
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[f][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int p = p0 + (wave + 4 * f) * 16 + lr;
    const int py = p >> a.lw, px = p & (W - 1);
    // the top left tap; a fragment beyond the tile reads the band's first pixel
    at[f] = lds + ((wave + 4 * f) * 16 < np ? (py - y0) * W2 + px : 0) * ps;
  }
  // Step ks from the fragments in wv[q], whose place the fragments of step ks + kConvSteps take.
  const auto product = [&](int q, int ks, const bf16x8* xv) {
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[f][n] = mfma(wv[q][n], xv[f], acc[f][n]);
    const bf16x8* next = a.wf + (size_t)min(ks + kConvSteps, steps - 1) * (NB * 64);
#pragma unroll
    for (int n = 0; n < NB; ++n) wv[q][n] = load_at<bf16x8>(next + n * 64, lane * 16);
  };
  bf16x8 xv[MF];
  if (a.lc >= 5) {
    // 32 input channels or more: a step lies within one tap, the same for all lanes
#pragma unroll
    for (int f = 0; f < MF; ++f) at[f] += 8 * lg;
    for (int ks0 = 0; ks0 < steps; ks0 += kConvSteps) {
#pragma unroll
      for (int q = 0; q < kConvSteps; ++q) {
        const int k0 = (ks0 + q) * 32, tap = k0 >> a.lc, ty = (tap * 11) >> 5;
        const int toff = (ty * W2 + tap - 3 * ty) * ps + (k0 & (a.cinp - 1));
#pragma unroll
        for (int f = 0; f < MF; ++f) xv[f] = *(const bf16x8*)(at[f] + toff);
        product(q, ks0 + q, xv);
      }
    }
  } else {
    for (int ks0 = 0; ks0 < steps; ks0 += kConvSteps) {
#pragma unroll
      for (int q = 0; q < kConvSteps; ++q) {
        const int k0 = (ks0 + q) * 32 + lg * 8, tap = k0 >> a.lc, ty = (tap * 11) >> 5, ch = k0 & (a.cinp - 1);
        const int toff = (ty * W2 + tap - 3 * ty) * ps + ch;
        // beyond the last tap (zero weights): the first row's left halo, which is zero
#pragma unroll
        for (int f = 0; f < MF; ++f) xv[f] = *(const bf16x8*)(tap < 9 ? at[f] + toff : lds + ch);
        product(q, ks0 + q, xv);
      }
    }
  }
  constexpr int C = NB * 16;
  f32x4 bias[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    bias[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (a.bias)
#pragma unroll
      for (int i = 0; i < 4; ++i) bias[n][i] = a.bias[n * 16 + 4 * lg + i];
  }
  const size_t pb = (size_t)b * npix + p0 + wave * 16 + lr;
  if (a.y) {
    float hw[NB][4][2];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        hw[n][i][0] = a.head[2 * (n * 16 + 4 * lg + i)];
        hw[n][i][1] = a.head[2 * (n * 16 + 4 * lg + i) + 1];
      }
    const float hb = a.head[2 * C + (lg & 1)];
#pragma unroll
    for (int f = 0; f < MF; ++f) {
      float h0 = 0.0f, h1 = 0.0f;
#pragma unroll
      for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float o = acc[f][n][i] + bias[n][i];
          const float v = (float)(bf16)(a.relu ? fmaxf(o, 0.0f) : o);
          h0 = fmaf(v, hw[n][i][0], h0);
          h1 = fmaf(v, hw[n][i][1], h1);
        }
      // lanes lr, lr + 16, lr + 32, lr + 48 hold the pixel's channels
#pragma unroll
      for (int m = 16; m < kWave; m <<= 1) {
        h0 += __shfl_xor(h0, m, kWave);
        h1 += __shfl_xor(h1, m, kWave);
      }
      if (lg < 2 && (wave + 4 * f) * 16 < np) a.y[2 * (pb + 64 * f) + lg] = (lg ? h1 : h0) + hb;
    }
    return;
  }
#pragma unroll
  for (int f = 0; f < MF; ++f) {
    if ((wave + 4 * f) * 16 >= np) continue;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const size_t o = (pb + 64 * f) * C + n * 16 + 4 * lg;
      f32x4 v = acc[f][n] + bias[n];
      if (a.relu)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.0f);
      if (a.out_bf) {
        bf16x4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (bf16)v[i];
        *(bf16x4*)(a.out_bf + o) = r;
      } else {
        *(f32x4*)(a.out_f + o) = v;
      }
    }
  }
}

template <int NB>
static hipError_t launch_conv_nb(const ConvArgs& a, int mf, dim3 grid, size_t lds, hipStream_t st) {
  switch (mf) {
    case 1: hipLaunchKernelGGL((conv3x3_kernel<NB, 1>), grid, dim3(kNetThreads), lds, st, a); break;
    case 2: hipLaunchKernelGGL((conv3x3_kernel<NB, 2>), grid, dim3(kNetThreads), lds, st, a); break;
    default: hipLaunchKernelGGL((conv3x3_kernel<NB, NB == 8 ? 2 : 4>), grid, dim3(kNetThreads), lds, st, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_conv(const ConvArgs& a, int batch, hipStream_t st) {
  const int npix = a.H * a.W;
  const int mf = conv_mf(a.H, a.W, a.cinp, a.nb, batch);
  const dim3 grid((npix + 64 * mf - 1) / (64 * mf), batch);
  const size_t lds = conv_lds_bytes(a.H, a.W, a.cinp, mf);
  // Layers whose weight fragments and two-fragment band exceed 160 KB (128 channels into 64) are refused as they were
  // when the weights lay in LDS beside the band; the kernel itself has room for them.
  const size_t weights = (size_t)a.ksteps * a.nb * kWave * sizeof(bf16x8);
  if (conv_lds_bytes(a.H, a.W, a.cinp, 2) + weights > 160 * 1024) return hipErrorInvalidValue;
  if (lds > 160 * 1024 || (1 << a.lc) != a.cinp || a.ksteps % kConvSteps || (a.mode == kUpCat && 2 * a.c1 != a.cinp))
    return hipErrorInvalidValue;
  switch (a.nb) {
    case 1: return launch_conv_nb<1>(a, mf, grid, lds, st);
    case 2: return launch_conv_nb<2>(a, mf, grid, lds, st);
    case 4: return launch_conv_nb<4>(a, mf, grid, lds, st);
    case 8: return launch_conv_nb<8>(a, mf, grid, lds, st);
    default: return hipErrorInvalidValue;
  }
}

// ---- weight gradient ----------------------------------------------------------------

namespace {

constexpr int kWgPix = 512;                // most pixels per band
constexpr int kWgChannels = 64;            // most input channels per workgroup
constexpr int kWgWaves = kNetThreads / kWave;
constexpr int kWgGroups = 512;             // most partials, and the floats they may hold together where
constexpr long long kWgFloats = 1 << 22;   // that leaves 128
constexpr size_t kWgLds = 80 * 1024;       // two workgroups per compute unit

typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

// Four rows of 16 channels (row-major in LDS, lane l % 16 gives the address of channels 4 (l % 4).. of
// row (l % 16) / 4) -> channel l % 16 of the four rows.
__device__ __forceinline__ bf16x4 read_columns(const bf16* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
}

__device__ __forceinline__ bf16x8 join8(bf16x4 lo, bf16x4 hi) {
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

int log2_of(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

// Bands of rows of a tile: the most rows (a power of two) whose pixels and staged operands keep
// within kWgPix and kWgLds.
struct WgradPlan {
  int rows, bands, groups, windows, lcg;
  size_t lds;
};

WgradPlan wgrad_plan(int H, int W, int cinp, int cout, int batch) {
  WgradPlan p{};
  const int cw = std::min(cinp, kWgChannels), blocks = (cw + 15) / 16;
  for (p.rows = H;; p.rows >>= 1) {
    const int npad = std::max(32, p.rows * W), staged = npad / W + 2;
    p.lds = ((size_t)staged * (W + 2) * (cw + 8) + (size_t)npad * (cout + 8)) * sizeof(bf16);
    if (p.rows == 1 || (p.rows * W <= kWgPix && p.lds <= kWgLds)) break;
  }
  // the sums over a band's slices, at the end
  p.lds = std::max(p.lds, (size_t)(kWgWaves - blocks) * 10 * kWave * sizeof(f32x4));
  p.bands = H / p.rows;
  const long long most = std::max<long long>(128, kWgFloats / (9LL * cinp * cout));
  p.groups = (int)std::min<long long>({(long long)batch * p.bands, (long long)kWgGroups, most});
  p.windows = (cinp + kWgChannels - 1) / kWgChannels;
  p.lcg = log2_of(cw / 8);
  return p;
}

}  // namespace

// part[g][tap cinp + ci][co] = sum_p in[p + off(tap)][ci] dz[p][co] over the pixels of the bands g, g + groups, ...
// of all tiles; bpart[g][co] = sum_p dz[p][co].  Grid: (groups, windows of 64 input channels).
//
// A workgroup stages a band of both operands pixel by pixel (16-byte copies, one pixel of halo) and reads
// them from LDS with transposing loads, which give a lane 4 pixels of its channel: a tap is an offset of whole
// pixels, so the 9 taps of a block of 16 input channels share the dz fragments and the addresses.  Wave w owns block
// w % blocks of the window with all 9 taps and all output channels in its accumulators (9 NB fragments);
// where there are fewer than 4 blocks the waves split the band's pixels and are added through LDS
// at the end.  The bias sums are one more product, with ones.
// Bound by the staging's latency (two workgroups per compute unit) and by LDS reads.  Batch 64 of
// 64 x 64 tiles, widths 16/32/64/64, seven layers: 1397 us with operands gathered element by
// element and one workgroup per tile, now 93.
template <int NB>
__global__ void __launch_bounds__(kNetThreads, 2) conv3x3_wgrad_kernel(ConvArgs a, const bf16* __restrict__ dz,
                                                                       int batch, int rows, int lcg,
                                                                       float* __restrict__ part,
                                                                       float* __restrict__ bpart) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int cout = NB * 16, ds = cout + 8;
  const int H = a.H, W = a.W, W2 = W + 2, npix = H * W;
  const int c0 = blockIdx.y * kWgChannels, cg = 1 << lcg, cw = 8 * cg, ps = cw + 8;
  const int np = rows * W, npad = max(32, np), staged = (npad >> a.lw) + 2, bands = H / rows;
  bf16* lin = (bf16*)smem;
  bf16* ldz = lin + (size_t)staged * W2 * ps;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lg = lane >> 4;
  const int blocks = (cw + 15) / 16, cb = wave % blocks, slice = wave / blocks, slices = kWgWaves / blocks;
  const bool bias = blockIdx.y == 0 && cb == 0;
  f32x4 acc[10][NB];
#pragma unroll
  for (int t = 0; t < 10; ++t)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;
#pragma unroll
  for (int i = 0; i < 8; ++i) ones[i] = (bf16)1.0f;
  // the halo columns are zero in every band
  for (int u = tid; u < staged * 2 * (cg + 1); u += kNetThreads) {
    const int g = u % (cg + 1), e = u / (cg + 1);
    *(bf16x8*)(lin + ((size_t)(e >> 1) * W2 + (e & 1) * (W + 1)) * ps + g * 8) = zero8();
  }
  for (int u = blockIdx.x; u < batch * bands; u += gridDim.x) {
    const int b = u / bands, y0 = (u - b * bands) * rows;
    const int nin = (staged << a.lw) << lcg, ndz = npad * (cout / 8);
    constexpr int kBatch = 4;
    for (int e0 = tid; e0 < nin; e0 += kNetThreads * kBatch) {
      bf16x8 v[kBatch];
#pragma unroll
      for (int q = 0; q < kBatch; ++q) {
        const int e = e0 + q * kNetThreads, g = e & (cg - 1), x = (e >> lcg) & (W - 1), y = y0 - 1 + (e >> lcg >> a.lw);
        v[q] = zero8();
        if (e < nin && y >= 0 && y < H) v[q] = load_input(a, b, y, x, c0 + g * 8);
      }
#pragma unroll
      for (int q = 0; q < kBatch; ++q) {
        const int e = e0 + q * kNetThreads, g = e & (cg - 1), x = (e >> lcg) & (W - 1), r = e >> lcg >> a.lw;
        if (e < nin) *(bf16x8*)(lin + ((size_t)r * W2 + x + 1) * ps + g * 8) = v[q];
      }
    }
    const bf16x8* src = (const bf16x8*)(dz + ((size_t)b * npix + (size_t)y0 * W) * cout);
    for (int e0 = tid; e0 < ndz; e0 += kNetThreads * kBatch) {
      bf16x8 v[kBatch];
#pragma unroll
      for (int q = 0; q < kBatch; ++q) {
        const int e = e0 + q * kNetThreads;
        v[q] = e < np * (cout / 8) ? src[e] : zero8();
      }
#pragma unroll
      for (int q = 0; q < kBatch; ++q) {
        const int e = e0 + q * kNetThreads;
        if (e < ndz) *(bf16x8*)(ldz + (e / (cout / 8)) * ds + (e % (cout / 8)) * 8) = v[q];
      }
    }
    __syncthreads();
    for (int s = 32 * slice; s < npad; s += 32 * slices) {
      const int q0 = s + 8 * lg + (lr >> 2), q1 = q0 + 4;
      const bf16* i0 = lin + ((q0 >> a.lw) * W2 + (q0 & (W - 1))) * ps + cb * 16 + 4 * (lr & 3);
      const bf16* i1 = lin + ((q1 >> a.lw) * W2 + (q1 & (W - 1))) * ps + cb * 16 + 4 * (lr & 3);
      const bf16* z0 = ldz + q0 * ds + 4 * (lr & 3);
      bf16x8 av[NB];
#pragma unroll
      for (int n = 0; n < NB; ++n) av[n] = join8(read_columns(z0 + 16 * n), read_columns(z0 + 4 * ds + 16 * n));
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int off = ((t / 3) * W2 + t % 3) * ps;
        const bf16x8 bv = join8(read_columns(i0 + off), read_columns(i1 + off));
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[t][n] = mfma(av[n], bv, acc[t][n]);
      }
      if (bias) {
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[9][n] = mfma(av[n], ones, acc[9][n]);
      }
    }
    __syncthreads();
  }
  if (slices > 1) {
    f32x4* red = (f32x4*)smem;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      if (slice > 0) {
#pragma unroll
        for (int t = 0; t < 10; ++t) red[((wave - blocks) * 10 + t) * kWave + lane] = acc[t][n];
      }
      __syncthreads();
      if (slice == 0) {
        for (int q = 1; q < slices; ++q)
#pragma unroll
          for (int t = 0; t < 10; ++t) acc[t][n] += red[((wave + (q - 1) * blocks) * 10 + t) * kWave + lane];
      }
      __syncthreads();
    }
  }
  if (slice > 0) return;
  // lane holds rows co = 16 n + 4 lg + i of column ci = 16 cb + lr
  const int ci = cb * 16 + lr, g = blockIdx.x;
  if (ci < cw) {
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int n = 0; n < NB; ++n)
        *(f32x4*)(part + ((size_t)(g * 9 + t) * a.cinp + c0 + ci) * cout + n * 16 + 4 * lg) = acc[t][n];
  }
  if (bias && lr == 0) {
#pragma unroll
    for (int n = 0; n < NB; ++n) *(f32x4*)(bpart + (size_t)g * cout + n * 16 + 4 * lg) = acc[9][n];
  }
}

int wgrad_partials(int H, int W, int cinp, int cout, int batch) { return wgrad_plan(H, W, cinp, cout, batch).groups; }

hipError_t launch_conv_wgrad(const ConvArgs& a, const bf16* dz, int cout, int batch, float* part, float* bpart,
                             hipStream_t st) {
  const WgradPlan p = wgrad_plan(a.H, a.W, a.cinp, cout, batch);
  if (p.lds > 160 * 1024) return hipErrorInvalidValue;
  const dim3 grid(p.groups, p.windows);
  switch (cout) {
    case 16:
      hipLaunchKernelGGL(conv3x3_wgrad_kernel<1>, grid, dim3(kNetThreads), p.lds, st, a, dz, batch, p.rows, p.lcg, part, bpart);
      break;
    case 32:
      hipLaunchKernelGGL(conv3x3_wgrad_kernel<2>, grid, dim3(kNetThreads), p.lds, st, a, dz, batch, p.rows, p.lcg, part, bpart);
      break;
    case 64:
      hipLaunchKernelGGL(conv3x3_wgrad_kernel<4>, grid, dim3(kNetThreads), p.lds, st, a, dz, batch, p.rows, p.lcg, part, bpart);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// gW[(tap cin + ci) cout + co] = sum_g part[g][tap cinp + ci][co];  gb[co] = sum_g bpart[g][co], for all
// layers in one launch (`taps` is 9 for 3x3 layers and 1 for the head, whose partials are [g][cin][cout]).
// One wave per slice of the partials, a lane per output: the loads of a slice are independent and
// coalesced over the lanes. Bound by latency: a launch per layer took 4.8 us each, 38 a gradient, all together now
// 14 (batch 64 of 64 x 64 tiles).
constexpr int kReduceSlices = 16;
__global__ void __launch_bounds__(kReduceSlices * kWave) wgrad_reduce_kernel(ReduceArgs a) {
  __shared__ float sums[kReduceSlices][kWave];
  int l = 0;
  while (l + 1 < kNetConv + 1 && (int)blockIdx.x >= a.l[l + 1].block) ++l;
  const ReduceLayer& L = a.l[l];
  const int lane = threadIdx.x % kWave, slice = threadIdx.x / kWave;
  const int nW = L.taps * L.cin * L.cout, idx = (blockIdx.x - L.block) * kWave + lane;
  const float* src = nullptr;
  long long stride = 0;
  if (idx < nW) {
    const int co = idx % L.cout, r = idx / L.cout, ci = r % L.cin, tap = r / L.cin;
    src = L.part + ((long long)tap * L.cinp + ci) * L.cout + co;
    stride = (long long)L.taps * L.cinp * L.cout;
  } else if (idx < nW + L.cout) {
    src = L.bpart + (idx - nW);
    stride = L.cout;
  }
  float s = 0.0f;
  if (src) {
#pragma unroll 8
    for (int g = slice; g < L.groups; g += kReduceSlices) s += src[g * stride];
  }
  sums[slice][lane] = s;
  __syncthreads();
  if (slice > 0 || !src) return;
  for (int q = 1; q < kReduceSlices; ++q) s += sums[q][lane];
  if (idx < nW) L.gW[idx] = s;
  else L.gb[idx - nW] = s;
}

hipError_t launch_wgrad_reduce(ReduceArgs a, hipStream_t st) {
  int blocks = 0;
  for (ReduceLayer& L : a.l) {
    L.block = blocks;
    blocks += (L.taps * L.cin * L.cout + L.cout + kWave - 1) / kWave;
  }
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(blocks), dim3(kReduceSlices * kWave), 0, st, a);
  return hipGetLastError();
}

// ---- weight fragments ------------------------------------------------------------

// Forward fragment e of lane l at (ks, nb): W[tap][ci][co] with k = 32 ks + 8 (l/16) + e =
// tap cinp + ci and co = 16 nb + l % 16 (0 for padded channels and taps >= 9).
// Data-gradient fragment: k' = tap' cout + co, n' = ci:  W[8 - tap'][ci][co].
__global__ void net_prepare_kernel(NetTable nt, const float* __restrict__ params, bf16x8* __restrict__ frags) {
  for (int li = 0; li < kNetConv; ++li) {
    const NetLayer& L = nt.l[li];
    const int nbf = L.cout / 16, nbb = L.cin / 16;
    const long long nf = (long long)L.ksteps * nbf * 64;
    const long long nbk = (li == 0) ? 0 : (long long)L.bksteps * nbb * 64;
    for (long long u = blockIdx.x * (long long)blockDim.x + threadIdx.x; u < nf + nbk;
         u += (long long)gridDim.x * blockDim.x) {
      bf16x8 v;
      if (u < nf) {
        const int lane = (int)(u % 64);
        const long long r = u / 64;
        const int nb = (int)(r % nbf), ks = (int)(r / nbf);
        const int co = nb * 16 + lane % 16;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = ks * 32 + 8 * (lane / 16) + e;
          const int tap = k / L.cinp, ci = k - tap * L.cinp;
          float w = 0.0f;
          if (tap < 9 && ci < L.cin) w = params[L.woff + ((long long)tap * L.cin + ci) * L.cout + co];
          v[e] = (bf16)w;
        }
        frags[L.ffrag + u] = v;
      } else {
        const long long ub = u - nf;
        const int lane = (int)(ub % 64);
        const long long r = ub / 64;
        const int nb = (int)(r % nbb), ks = (int)(r / nbb);
        const int ci = nb * 16 + lane % 16;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = ks * 32 + 8 * (lane / 16) + e;
          const int tap = k / L.cout, co = k - tap * L.cout;
          float w = 0.0f;
          if (tap < 9) w = params[L.woff + ((long long)(8 - tap) * L.cin + ci) * L.cout + co];
          v[e] = (bf16)w;
        }
        frags[L.bfrag + ub] = v;
      }
    }
  }
}

hipError_t launch_net_prepare(const NetTable& nt, const float* params, bf16x8* frags, hipStream_t st) {
  hipLaunchKernelGGL(net_prepare_kernel, dim3(256), dim3(256), 0, st, nt, params, frags);
  return hipGetLastError();
}

// ---- gradient routing between levels ----------------------------------------------------

// Grid: (units of 8 channels of a tile / 256, batch). Bound by latency and its reads, up to 6 fp32 values per
// output: one element per thread, with 64-bit divisions for its place, took 17 us at the largest level of 64
// tiles of 64 x 64, now 10.
__global__ void __launch_bounds__(kNetThreads) route_kernel(RouteArgs a) {
  const int u = blockIdx.x * kNetThreads + threadIdx.x, npix = a.H * a.W;
  if (u >= npix << a.lcg) return;
  const int c = (u & ((1 << a.lcg) - 1)) * 8, p = u >> a.lcg, x = p & (a.W - 1), y = p >> a.lw;
  const size_t b = blockIdx.y, pix = b * npix + p;
  const bf16x8 act = *(const bf16x8*)(a.act + (pix << (a.lcg + 3)) + c);
  f32x4 g[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  if (a.fine) {
    const float* f = a.fine + (4 * b * npix + 4 * y * a.W + 2 * x) * a.fstride + a.foff + c;
    const float* d = f + (size_t)2 * a.W * a.fstride;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      g[h] += (*(const f32x4*)(f + 4 * h) + *(const f32x4*)(f + a.fstride + 4 * h)) +
              (*(const f32x4*)(d + 4 * h) + *(const f32x4*)(d + a.fstride + 4 * h));
  }
  if (a.same) {
    const float* f = a.same + pix * a.sstride + a.soff + c;
#pragma unroll
    for (int h = 0; h < 2; ++h) g[h] += *(const f32x4*)(f + 4 * h);
  }
  if (a.coarse) {
    const float* f = a.coarse + (b * (npix >> 2) + (y >> 1) * (a.W >> 1) + (x >> 1)) * a.cstride + c;
#pragma unroll
    for (int h = 0; h < 2; ++h) g[h] += 0.25f * *(const f32x4*)(f + 4 * h);
  }
  bf16x8 o;
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = (float)act[i] > 0.0f ? (bf16)g[i / 4][i % 4] : (bf16)0.0f;
  *(bf16x8*)(a.dz + (pix << (a.lcg + 3)) + c) = o;
}

hipError_t launch_route(const RouteArgs& a, int batch, hipStream_t st) {
  const int units = a.H * a.W << a.lcg;
  hipLaunchKernelGGL(route_kernel, dim3((units + kNetThreads - 1) / kNetThreads, batch), dim3(kNetThreads), 0, st, a);
  return hipGetLastError();
}

// ---- head: 1x1 output layer, loss, and the first backward steps ----------------------------

namespace {

__device__ __forceinline__ double block_sum_d(double v, double* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < kNetThreads / kWave; ++w) s += red[w];
  return s;
}

// (B v)_p for node p = (li, lj) of the tile operator; v at p's place in LDS rows of stride T + 2, zero
// where there is no node.
__device__ __forceinline__ cplx<float> tile_apply(const cplx<float>* tab, const TileDescDev& d, int li, int lj,
                                                  const cplx<float>* v, int stride) {
  const int xc = (li == 0 && (d.edges & 1)) ? 0 : ((li == d.nx - 1 && (d.edges & 2)) ? 2 : 1);
  const int yc = (lj == 0 && (d.edges & 4)) ? 0 : ((lj == d.ny - 1 && (d.edges & 8)) ? 2 : 1);
  const cplx<float>* c = tab + kStencilPts * (3 * yc + xc);
  cplx<float> acc = c[kC] * v[0];
  acc = cfma(c[kW], v[-1], acc);
  acc = cfma(c[kE], v[1], acc);
  acc = cfma(c[kS], v[-stride], acc);
  acc = cfma(c[kSW], v[-stride - 1], acc);
  acc = cfma(c[kN], v[stride], acc);
  return cfma(c[kNE], v[stride + 1], acc);
}

__device__ __forceinline__ void zero_sides(cplx<float>* f, int rows, int T) {
  for (int u = threadIdx.x; u < 2 * rows; u += kNetThreads) f[(u >> 1) * (T + 2) + (u & 1) * (T + 1)] = czero<float>();
}

}  // namespace

// The loss of tile b, with e = m (y - t) and r = B e (y = a7 W8 + b8, B the tile's subdomain operator, m its
// node mask), and its gradient:
//   loss_b = w_res ||r||^2 / ||B t||^2 + w_err ||e||^2 / ||m t||^2,
//   dL/dy  = (w_res 2 B^H r / ||B t||^2 + w_err 2 e / ||m t||^2) / batch   on nodes,
// then the head's weight and bias partials and dz7 = (dL/dy W8^T) * (a7 > 0).
//
// The denominators depend on the target alone, so a first launch sums them and the second one needs
// no other sum over a tile: both take strips of kHeadRows rows, and the second forms e on two and r on one more
// row to each side itself. One workgroup per tile, with e and r in global memory, was a chain of
// three passes on a quarter of the chip: 125 us for 64 tiles of 64 x 64, both launches now 18.
//
// den[b][strip] = (||m t||^2, ||B t||^2) over the strip.  Grid: (T / kHeadRows, batch).
__global__ void __launch_bounds__(kNetThreads) head_norms_kernel(HeadArgs a) {
  __shared__ cplx<float> tab[kClasses * kStencilPts];
  __shared__ double red[kNetThreads / kWave];
  __shared__ cplx<float> f[(kHeadRows + 2) * (kMaxTile + 2)];
  const int b = blockIdx.y, T = a.T, lt = a.lt, S = T + 2, y0 = blockIdx.x * kHeadRows;
  const TileDescDev d = a.desc[b];
  build_class_table<float>(d.robin, d.kh, d.kh * d.kh, tab);
  zero_sides(f, kHeadRows + 2, T);
  const float* t = a.t + ((size_t)b << (2 * lt + 1));
  double err = 0.0, res = 0.0;
  for (int u = threadIdx.x; u < (kHeadRows + 2) << lt; u += kNetThreads) {
    const int r = u >> lt, li = u & (T - 1), lj = y0 - 1 + r;
    cplx<float> v = czero<float>();
    if (li < d.nx && lj >= 0 && lj < d.ny) v = cplx<float>{t[2 * (lj * T + li)], t[2 * (lj * T + li) + 1]};
    f[r * S + li + 1] = v;
    if (r >= 1 && r <= kHeadRows) err += (double)v.re * v.re + (double)v.im * v.im;
  }
  __syncthreads();
  for (int u = threadIdx.x; u < kHeadRows << lt; u += kNetThreads) {
    const int r = u >> lt, li = u & (T - 1), lj = y0 + r;
    if (li < d.nx && lj < d.ny) res += (double)cabs2(tile_apply(tab, d, li, lj, f + (r + 1) * S + li + 1, S));
  }
  err = block_sum_d(err, red);
  res = block_sum_d(res, red);
  if (threadIdx.x == 0) {
    double* o = a.den + 2 * ((size_t)b * gridDim.x + blockIdx.x);
    o[0] = err;
    o[1] = res;
  }
}

// loss, part and bpart: one value or row per strip.  Grid: (T / kHeadRows, batch).
template <int C>
__global__ void __launch_bounds__(kNetThreads) head_kernel(HeadArgs a) {
  __shared__ cplx<float> tab[kClasses * kStencilPts];
  __shared__ double red[kNetThreads / kWave];
  __shared__ float hw[C * 2 + 2];
  __shared__ float pred[kNetThreads / kWave][C * 2 + 2];
  __shared__ cplx<float> E[(kHeadRows + 4) * (kMaxTile + 2)];
  __shared__ cplx<float> R[(kHeadRows + 2) * (kMaxTile + 2)];
  const int b = blockIdx.y, tid = threadIdx.x, T = a.T, lt = a.lt, S = T + 2, y0 = blockIdx.x * kHeadRows;
  const size_t strip = (size_t)b * gridDim.x + blockIdx.x;
  for (int i = tid; i < 2 * C + 2; i += kNetThreads)
    hw[i] = i < 2 * C ? a.params[a.woff + i] : a.params[a.boff + i - 2 * C];
  const TileDescDev d = a.desc[b];
  build_class_table<float>(d.robin, d.kh, d.kh * d.kh, tab);
  zero_sides(E, kHeadRows + 4, T);
  zero_sides(R, kHeadRows + 2, T);
  double den_err = 0.0, den_res = 0.0;
  for (unsigned s = 0; s < gridDim.x; ++s) {
    den_err += a.den[2 * ((size_t)b * gridDim.x + s)];
    den_res += a.den[2 * ((size_t)b * gridDim.x + s) + 1];
  }
  if (den_err <= 0.0) den_err = 1.0;
  if (den_res <= 0.0) den_res = 1.0;
  __syncthreads();
  const bf16* act = a.a7 + ((size_t)b << (2 * lt)) * C;
  const float* t = a.t + ((size_t)b << (2 * lt + 1));
  double num_err = 0.0, num_res = 0.0;
  for (int u = tid; u < (kHeadRows + 4) << lt; u += kNetThreads) {
    const int r = u >> lt, li = u & (T - 1), lj = y0 - 2 + r, p = lj * T + li;
    cplx<float> e = czero<float>();
    if (li < d.nx && lj >= 0 && lj < d.ny) {
      float v0 = hw[2 * C], v1 = hw[2 * C + 1];
#pragma unroll
      for (int c8 = 0; c8 < C / 8; ++c8) {
        const bf16x8 av = *(const bf16x8*)(act + (size_t)p * C + 8 * c8);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          v0 = fmaf((float)av[i], hw[2 * (8 * c8 + i)], v0);
          v1 = fmaf((float)av[i], hw[2 * (8 * c8 + i) + 1], v1);
        }
      }
      e = cplx<float>{v0 - t[2 * p], v1 - t[2 * p + 1]};
    }
    E[r * S + li + 1] = e;
    if (r >= 2 && r < kHeadRows + 2) num_err += (double)e.re * e.re + (double)e.im * e.im;
  }
  __syncthreads();
  // R holds conj(r): B^H r = conj(B conj(r)) (B is complex symmetric)
  for (int u = tid; u < (kHeadRows + 2) << lt; u += kNetThreads) {
    const int r = u >> lt, li = u & (T - 1), lj = y0 - 1 + r;
    cplx<float> v = czero<float>();
    if (li < d.nx && lj >= 0 && lj < d.ny) v = tile_apply(tab, d, li, lj, E + (r + 1) * S + li + 1, S);
    R[r * S + li + 1] = cplx<float>{v.re, -v.im};
    if (r >= 1 && r <= kHeadRows) num_res += (double)cabs2(v);
  }
  __syncthreads();
  const float sres = (float)(2.0 * a.w_res / (den_res * a.batch));
  const float serr = (float)(2.0 * a.w_err / (den_err * a.batch));
  float pw[C * 2 + 2];
#pragma unroll
  for (int i = 0; i < 2 * C + 2; ++i) pw[i] = 0.0f;
  bf16* dz = a.dz7 + ((size_t)b << (2 * lt)) * C;
  for (int u = tid; u < kHeadRows << lt; u += kNetThreads) {
    const int r = u >> lt, li = u & (T - 1), lj = y0 + r, p = lj * T + li;
    float g0 = 0.0f, g1 = 0.0f;
    if (li < d.nx && lj < d.ny) {
      const cplx<float> q = tile_apply(tab, d, li, lj, R + (r + 1) * S + li + 1, S);
      const cplx<float> e = E[(r + 2) * S + li + 1];
      g0 = sres * q.re + serr * e.re;
      g1 = -sres * q.im + serr * e.im;
    }
    pw[2 * C] += g0;
    pw[2 * C + 1] += g1;
#pragma unroll
    for (int c8 = 0; c8 < C / 8; ++c8) {
      const bf16x8 av = *(const bf16x8*)(act + (size_t)p * C + 8 * c8);
      bf16x8 o;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = 8 * c8 + i;
        const float v = (float)av[i];
        pw[2 * c] = fmaf(v, g0, pw[2 * c]);
        pw[2 * c + 1] = fmaf(v, g1, pw[2 * c + 1]);
        o[i] = v > 0.0f ? (bf16)(g0 * hw[2 * c] + g1 * hw[2 * c + 1]) : (bf16)0.0f;
      }
      *(bf16x8*)(dz + (size_t)p * C + 8 * c8) = o;
    }
  }
  num_err = block_sum_d(num_err, red);
  num_res = block_sum_d(num_res, red);
  if (tid == 0) a.loss[strip] = a.w_res * num_res / den_res + a.w_err * num_err / den_err;
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int i = 0; i < 2 * C + 2; ++i) {
    const float s = wave_total(pw[i]);
    if (lane == kWave - 1) pred[wave][i] = s;
  }
  __syncthreads();
  for (int i = tid; i < 2 * C + 2; i += kNetThreads) {
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < kNetThreads / kWave; ++w) s += pred[w][i];
    if (i < 2 * C) a.part[strip * 2 * C + i] = s;
    else a.bpart[strip * 2 + i - 2 * C] = s;
  }
}

hipError_t launch_head(const HeadArgs& a, hipStream_t st) {
  const dim3 grid(head_strips(a.T), a.batch);
  hipLaunchKernelGGL(head_norms_kernel, grid, dim3(kNetThreads), 0, st, a);
  switch (a.c1) {
    case 16: hipLaunchKernelGGL(head_kernel<16>, grid, dim3(kNetThreads), 0, st, a); break;
    case 32: hipLaunchKernelGGL(head_kernel<32>, grid, dim3(kNetThreads), 0, st, a); break;
    case 64: hipLaunchKernelGGL(head_kernel<64>, grid, dim3(kNetThreads), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---- optimiser -----------------------------------------------------------------------

// Adam (Kingma and Ba, 2015); c1 = 1 - beta1^t, c2 = 1 - beta2^t.
__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, long long n, float lr, float b1, float b2, float eps, float c1,
                            float c2) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, long long n, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t st) {
  const int blocks = (int)std::min<long long>((n + 255) / 256, 1024);
  hipLaunchKernelGGL(adam_kernel, dim3(blocks), dim3(256), 0, st, p, g, m, v, n, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

// ---- tiles ---------------------------------------------------------------------------

// Network input of solve (rhs, sub) = tile rhs * nsub + sub, from f = R_j r.
__global__ void __launch_bounds__(kNetThreads) tiles_kernel(TileArgs a) {
  __shared__ double red[kNetThreads / kWave];
  const int nsub = a.cs.nsub;
  const int b = blockIdx.x, rhs = b / nsub, sub = b - rhs * nsub;
  if (a.done && a.done[rhs]) return;
  const SubDesc d = a.subs[sub];
  const int T = a.T, nx = d.nx, nj = d.nx * d.ny, ldg = a.cs.n - 1;
  const long long jstep = a.jdev ? (long long)*a.jdev : 0;
  const cplx<double>* r = a.r + jstep * a.rslot + (long long)rhs * a.rstride;
  double s2 = 0.0;
  for (int n = threadIdx.x; n < nj; n += kNetThreads) {
    const int lj = n / nx, li = n - lj * nx;
    s2 += cabs2(r[(long long)(d.j0 + lj - 1) * ldg + (d.i0 + li - 1)]);
  }
  s2 = block_sum_d(s2, red);
  const double fn = sqrt(s2);
  const double s = fn > 0.0 ? sqrt((double)nj) / fn : 0.0;
  if (threadIdx.x == 0) a.scale[b] = s;
  const float kh = (float)a.cs.kh;
  for (int p = threadIdx.x; p < T * T; p += kNetThreads) {
    const int li = p % T, lj = p / T;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (li < d.nx && lj < d.ny) {
      const cplx<double> f = r[(long long)(d.j0 + lj - 1) * ldg + (d.i0 + li - 1)];
      const int cls = node_class(d.i0 + li, d.j0 + lj, d.ax, d.bx, d.ay, d.by);
      const int xc = cls % 3, yc = cls / 3;
      const bool imp = (xc == 0 && (d.robin & 1)) || (xc == 2 && (d.robin & 2)) || (yc == 0 && (d.robin & 4)) ||
                       (yc == 2 && (d.robin & 8));
      v[0] = (float)(s * f.re);
      v[1] = (float)(s * f.im);
      v[2] = kh;
      v[3] = imp ? -1.0f : 1.0f;
    }
    const size_t q = (size_t)b * T * T + p;
    if (a.xb) {
      bf16x8 o = zero8();
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = (bf16)v[i];
      *(bf16x8*)(a.xb + 8 * q) = o;
    }
    if (a.xf) *(f32x4*)(a.xf + 4 * q) = f32x4{v[0], v[1], v[2], v[3]};
  }
}

hipError_t launch_tiles(const TileArgs& a, int nsub, int nrhs, hipStream_t st) {
  hipLaunchKernelGGL(tiles_kernel, dim3(nsub * nrhs), dim3(kNetThreads), 0, st, a);
  return hipGetLastError();
}

// t[b][lj][li] = scale[b] * u[rhs][off + lj nx + li] on nodes, 0 elsewhere.
__global__ void packed_to_tiles_kernel(const SubDesc* __restrict__ subs, int nsub, long long nfine,
                                       const cplx<double>* __restrict__ u, const double* __restrict__ scale, int T,
                                       float* __restrict__ t) {
  const int b = blockIdx.x, rhs = b / nsub, sub = b - rhs * nsub;
  const SubDesc d = subs[sub];
  const double s = scale[b];
  for (int p = threadIdx.x; p < T * T; p += blockDim.x) {
    const int li = p % T, lj = p / T;
    float v0 = 0.f, v1 = 0.f;
    if (li < d.nx && lj < d.ny) {
      const cplx<double> x = u[(long long)rhs * nfine + d.off + (long long)lj * d.nx + li];
      v0 = (float)(s * x.re);
      v1 = (float)(s * x.im);
    }
    t[((size_t)b * T * T + p) * 2] = v0;
    t[((size_t)b * T * T + p) * 2 + 1] = v1;
  }
}

hipError_t launch_packed_to_tiles(const SubDesc* subs, int nsub, int nrhs, long long nfine,
                                  const cplx<double>* u, const double* scale, int T, float* t, hipStream_t st) {
  hipLaunchKernelGGL(packed_to_tiles_kernel, dim3(nsub * nrhs), dim3(256), 0, st, subs, nsub, nfine, u, scale, T, t);
  return hipGetLastError();
}

hipError_t configure_net() {
  const void* kernels[] = {
      (const void*)conv3x3_kernel<1, 1>, (const void*)conv3x3_kernel<1, 2>, (const void*)conv3x3_kernel<1, 4>,
      (const void*)conv3x3_kernel<2, 1>, (const void*)conv3x3_kernel<2, 2>, (const void*)conv3x3_kernel<2, 4>,
      (const void*)conv3x3_kernel<4, 1>, (const void*)conv3x3_kernel<4, 2>, (const void*)conv3x3_kernel<4, 4>,
      (const void*)conv3x3_kernel<8, 1>, (const void*)conv3x3_kernel<8, 2>,
      (const void*)conv3x3_wgrad_kernel<1>, (const void*)conv3x3_wgrad_kernel<2>, (const void*)conv3x3_wgrad_kernel<4>};
  for (const void* k : kernels)
    if (hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)) return e;
  return hipSuccess;
}

}  // namespace ddh
