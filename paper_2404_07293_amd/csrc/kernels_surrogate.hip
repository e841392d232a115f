// Kernels of the spectral-convolution surrogate: the lift, the fused halves of
// a Fourier layer and its per-mode mixing, the head and the Adam update. The
// FP32 backward pass runs the same kernels with the adjoint tables and
// weights (the remaining backward kernels are in kernels_surrogate_bwd.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "scw_internal.h"
#include "surrogate_device.h"

namespace scw {
namespace {

__global__ void adam(float* p, const float* g, float* m, float* v, long long n, float lr,
                     float b1, float b2, float eps, float c1, float c2) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---------------------------------------------------------------- fused Fourier layer
// The two halves of one Fourier layer around its per-mode mixing (which stays
// a batched product over the patches, so that each mode's 32 x 32 weights are
// read once per tile of patches rather than once per patch):
//   forward  H[b][i][ky][kx] = sum_y fy[ky][y] sum_x h[b][i][y][x] fx[x][kx]
//   inverse  z[b][o][y][x] = Re sum_kx (sum_ky iy[y][ky] G[b][o][ky][kx]) ix[kx][x]
//                          + sum_i pw[i][o] h[b][i][y][x] + pb[o]
//            h'[b][o] = GELU(z[b][o]) (or z itself after the last layer)
// With BF16, both operands of every product are rounded to bf16 (nearest
// even) first, as the matrix-core products of the unfused path round them;
// sums stay FP32.
// Truncated forward DFT of 8 channels of one patch per block:
//   out[b][i][ky][kx] = sum_y fy[ky][y] sum_x h[b][i][y][x] fx[x][kx]
// (KY x KX modes; fy is [KY][32], fx is [32][KX], both complex). Grid (4, B),
// 256 T threads. Thread (c, y) = (t / 32 % 8, t % 32) first transforms row y of
// channel c in registers, for the t / 256-th T-th of the kx; the column transform
// then runs over (c, mode). T = 2 while there is at most one block per CU, where
// each thread's chain of sums is what takes the time (64 patches in bf16
// products: 11.4 us with T = 1, 9.8 with T = 2).
// MM selects the mode-major output layout [mode][b][i] (a Fourier layer's
// spectra, read per mode by the mixing); otherwise [b][i][mode] (the head).
template <bool BF16, int KY, int KX, bool MM, int T>
__global__ void __launch_bounds__(256 * T) fused_dft_fwd(const float* __restrict__ h,
                                                     const f2* __restrict__ fy,
                                                     const f2* __restrict__ fx,
                                                     f2* __restrict__ H) {
  // Padded strides against LDS bank conflicts (16 lanes of 8 bytes per
  // cycle): a channel's rows start 2 (mod 16) complex values apart, so that 8
  // channels x 2 consecutive kx hit distinct banks; the ky rows of fy are 33
  // apart, so that a wave reading two ky groups hits two banks.
  constexpr int HXS = SN * KX + 2, FYS = SN + 1;
  __shared__ f2 hx[8 * HXS];
  __shared__ f2 fys[KY * FYS], fxs[SN * KX];
  const int t = threadIdx.x, b = blockIdx.y, c0 = blockIdx.x * 8;
  const int c = (t >> 5) & 7, y = t & 31;
  const int part = __builtin_amdgcn_readfirstlane(t >> 8);
  const int kx0 = KX * part / T, kx1 = KX * (part + 1) / T;
  float row[SN];
  const float4* src =
      reinterpret_cast<const float4*>(h + (((long long)b * SW + c0 + c) * SN + y) * SN);
  // all loads go out before the first is waited for (tables past their end read
  // the last entry again)
  constexpr int NY = (KY * SN + 256 * T - 1) / (256 * T), NX = (SN * KX + 256 * T - 1) / (256 * T);
  float4 rv[SN / 4];
  f2 yv[NY], xv[NX];
#pragma unroll
  for (int q = 0; q < SN / 4; ++q) rv[q] = src[q];
#pragma unroll
  for (int k = 0; k < NY; ++k) yv[k] = fy[min(t + 256 * T * k, KY * SN - 1)];
  if (BF16)
#pragma unroll
    for (int k = 0; k < NX; ++k) xv[k] = fx[min(t + 256 * T * k, SN * KX - 1)];
#pragma unroll
  for (int q = 0; q < SN / 4; ++q) {
    row[4 * q] = op<BF16>(rv[q].x);
    row[4 * q + 1] = op<BF16>(rv[q].y);
    row[4 * q + 2] = op<BF16>(rv[q].z);
    row[4 * q + 3] = op<BF16>(rv[q].w);
  }
#pragma unroll
  for (int k = 0; k < NY; ++k) {
    const int i = min(t + 256 * T * k, KY * SN - 1);
    fys[(i / SN) * FYS + i % SN] = op<BF16>(yv[k]);
  }
  if (BF16)
#pragma unroll
    for (int k = 0; k < NX; ++k) fxs[min(t + 256 * T * k, SN * KX - 1)] = op<BF16>(xv[k]);
  __syncthreads();
  if constexpr (BF16) {  // every product of two rounded operands, as defined
#pragma unroll 3
    for (int kx = kx0; kx < kx1; ++kx) {
      float re = 0.f, im = 0.f;
#pragma unroll
      for (int x = 0; x < SN; ++x) {
        const f2 w = fxs[x * KX + kx];
        re = fmaf(row[x], w.x, re);
        im = fmaf(row[x], w.y, im);
      }
      hx[c * HXS + y * KX + kx] = op<BF16>(f2{re, im});
    }
  } else {
    // The twiddles of x and 32 - x are conjugate: with s = row[x] + row[32-x]
    // and d = row[x] - row[32-x], the pair adds s Re w to the real part and
    // d Im w to the imaginary part (x = 0 and 16 stand alone; a layer's table
    // holds kx = 0..8, the head's kx = -7..7 scaled by 1/32, both conjugate
    // symmetric). The index is wave-uniform, so the twiddles come through the
    // scalar cache.
    float sx[SN / 2], dx[SN / 2];
#pragma unroll
    for (int x = 1; x < SN / 2; ++x) {
      sx[x] = row[x] + row[SN - x];
      dx[x] = row[x] - row[SN - x];
    }
#pragma unroll 3
    for (int kx = kx0; kx < kx1; ++kx) {
      const f2 w0 = fx[kx], w16 = fx[(SN / 2) * KX + kx];
      float re = fmaf(row[0], w0.x, row[SN / 2] * w16.x);
      float im = fmaf(row[0], w0.y, row[SN / 2] * w16.y);
#pragma unroll
      for (int x = 1; x < SN / 2; ++x) {
        const f2 w = fx[x * KX + kx];
        re = fmaf(sx[x], w.x, re);
        im = fmaf(dx[x], w.y, im);
      }
      hx[c * HXS + y * KX + kx] = f2{re, im};
    }
  }
  __syncthreads();
  // column transform: items (ky group of KG, kx, channel), channel fastest;
  // each hx value read serves KG modes
  constexpr int NMODE = KY * KX;
  constexpr int KG = 3, NKG = (KY + KG - 1) / KG;
  for (int i = t; i < 8 * KX * NKG; i += 256 * T) {
    const int cc = i % 8, kx = (i / 8) % KX, g = i / (8 * KX);
    float re[KG], im[KG];
#pragma unroll
    for (int j = 0; j < KG; ++j) re[j] = im[j] = 0.f;
    const f2* hc = hx + cc * HXS + kx;  // hc[yy * KX]
    if constexpr (BF16) {
#pragma unroll 4
      for (int yy = 0; yy < SN; ++yy) {
        const f2 v = hc[yy * KX];
#pragma unroll
        for (int j = 0; j < KG; ++j) {
          const f2 a = fys[min(g * KG + j, KY - 1) * FYS + yy];
          re[j] = fmaf(a.x, v.x, fmaf(-a.y, v.y, re[j]));
          im[j] = fmaf(a.x, v.y, fmaf(a.y, v.x, im[j]));
        }
      }
    } else {
      // rows yy and 32 - yy have conjugate twiddles: w a + conj(w) b =
      // Re w (a + b) + i Im w (a - b); rows 0 and 16 stand alone
#pragma unroll
      for (int yy = 0; yy <= SN / 2; yy += SN / 2) {
        const f2 v = hc[yy * KX];
#pragma unroll
        for (int j = 0; j < KG; ++j) {
          const f2 a = fys[min(g * KG + j, KY - 1) * FYS + yy];
          re[j] = fmaf(a.x, v.x, fmaf(-a.y, v.y, re[j]));
          im[j] = fmaf(a.x, v.y, fmaf(a.y, v.x, im[j]));
        }
      }
#pragma unroll 3
      for (int yy = 1; yy < SN / 2; ++yy) {
        const f2 va = hc[yy * KX], vb = hc[(SN - yy) * KX];
        const f2 p = f2{va.x + vb.x, va.y + vb.y}, q = f2{va.x - vb.x, va.y - vb.y};
#pragma unroll
        for (int j = 0; j < KG; ++j) {
          const f2 a = fys[min(g * KG + j, KY - 1) * FYS + yy];
          re[j] = fmaf(a.x, p.x, fmaf(-a.y, q.y, re[j]));
          im[j] = fmaf(a.x, p.y, fmaf(a.y, q.x, im[j]));
        }
      }
    }
#pragma unroll
    for (int j = 0; j < KG; ++j) {
      const int ky = g * KG + j;
      if (ky >= KY) break;
      const int m = ky * KX + kx;
      if (MM)
        H[((long long)m * gridDim.y + b) * SW + c0 + cc] = f2{re[j], im[j]};
      else
        H[((long long)b * SW + c0 + cc) * NMODE + m] = f2{re[j], im[j]};
    }
  }
}

// GELU(z) = z (1 + erf(z / sqrt 2)) / 2 for the forward pass, with erf from
// Abramowitz and Stegun 7.1.26 (Hastings' rational approximation, absolute
// error at most 1.5e-7): erf(x) = 1 - t (a1 + t (a2 + ... + t a5)) e^{-x^2},
// t = 1 / (1 + p x), x >= 0. Branch-free: one reciprocal and one exponential.
// For z < 0, 1 + erf(z / sqrt 2) is formed directly as the product, without
// the cancellation of 1 - (1 - product).
__device__ __forceinline__ float gelu_fwd_f(float z) {
  const float x = fabsf(z) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.f));
  float q = fmaf(1.061405429f, t, -1.453152027f);
  q = fmaf(q, t, 1.421413741f);
  q = fmaf(q, t, -0.284496736f);
  q = fmaf(q, t, 0.254829592f);
  const float pe = q * t * __expf(-x * x);  // 1 - erf(x)
  return 0.5f * z * (z >= 0.f ? 2.f - pe : pe);
}

// The same inverse half of a Fourier layer with its two dense parts on the
// matrix cores. For one patch and image row y, the 32 outputs x 32 pixels
//   z[o][y][x] = sum_i pw[i][o] h[i][y][x]
//              + sum_kx (Re gy[o][y][kx] Re ix[kx][x] - Im gy[o][y][kx] Im ix[kx][x])
//              + pb[o]
// are one 32 x 32 FP32 tile with K = 32 + 18: the pointwise weights and the
// row transform's twiddles are fixed operands held in registers, the pixels
// come straight from memory (32 consecutive x per half-wave) and the column
// transform gy[o][y][kx] = sum_ky iy[y][ky] G[o][ky][kx] is formed on the
// vector units, 8 rows at a time, into LDS. The rows y and 32 - y have
// conjugate twiddles, so one set of products gives both: with A = sum Re iy G
// and B = sum Im iy G, gy[y] = A + i B and gy[32 - y] = A - i B (per complex
// part below); each group of 8 rows is 4 such pairs (rows 0 and 16 use direct
// sums). With BF16 these are still products of two rounded operands: rounding
// to nearest even is symmetric, so the rounded twiddles of 32 - y remain the
// conjugates of those of y.
// One patch per block of 8 waves; wave w takes slot w of each group, and its
// pixel loads for the next group are issued once the current ones are used.
// Grid (B, splits): a block runs 4 / splits of the four row groups, so that a
// batch of few patches still reaches many CUs (each block stages G again).
//
// The same kernel is the adjoint of the forward half in the FP32 backward
// pass, because the adjoint of a truncated DFT is an inverse transform with
// conjugate tables:
//   INV_ADJOINT  out[b][i] = (Re fy^H gH fx^H + sum_o pw[i][o] gz[b][o]) GELU'(zp)
//                (G = gH, h = gz, the weights read transposed, no bias; zp is
//                the previous layer's pre-activation, or null for the lift)
//   INV_HEAD     out[b][i] = Re hy^H gF hx^H with gF[b][m][i] =
//                sum_c gout[b][c][m] conj(head[i][c][m]) formed while staging
constexpr int INVM_T = 512;
enum { INV_LAYER = 0, INV_ADJOINT = 1, INV_HEAD = 2 };
// The image rows of group k (0..3), slot w (0..7): conjugate pairs (y, 32 - y)
// in slots w and w + 4, y = 4k + 1 + (w mod 4); the last group's slots 3 and
// 7 hold the self-paired rows 0 and 16.
__device__ __forceinline__ int inv_row(int k, int w) {
  const int base = 4 * k + 1 + (w & 3);
  if (k == 3 && (w & 3) == 3) return w < 4 ? 0 : SN / 2;
  return w < 4 ? base : SN - base;
}
// NT: pixels and outputs non-temporal (batches past the last-level cache: 4096
// patches 351 us, 367 without).
template <bool BF16, int MODE, bool NT = false>
__global__ void __launch_bounds__(INVM_T) __attribute__((amdgpu_waves_per_eu(4)))
fused_dft_inv_mfma(
    const f2* __restrict__ G, const float* __restrict__ h, const f2* __restrict__ iy,
    const f2* __restrict__ ix, const float* __restrict__ pw, const float* __restrict__ pb,
    float* __restrict__ z_out, float* __restrict__ h_out, int apply_gelu,
    const float* __restrict__ zp) {
  constexpr int KY = MODE == INV_HEAD ? 15 : SKY, KX = MODE == INV_HEAD ? 15 : SKX;
  constexpr int GYS = 2 * KX + 1;         // gy row stride (floats), odd against bank conflicts
  constexpr int GS = MODE == INV_HEAD ? SW + 1 : SW;  // the head writes gsm along modes
  __shared__ f2 gsm[KY * KX][GS];         // the patch's G, [mode][o]
  __shared__ f2 iys[SN * KY];             // [y][ky]
  __shared__ float gyl[8][SW][GYS];       // [row of the group][o][kx re | kx im]
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, li = lane & 31, lh = lane >> 5;
  const int b = blockIdx.x;
  const int groups = (SN / 8) / gridDim.y, g0 = blockIdx.y * groups;
  if constexpr (MODE == INV_HEAD) {
    constexpr int NMODE = KY * KX, OUT = 3;
    const f2* go = G + (long long)b * OUT * NMODE;        // gout[b]
    const f2* wh = reinterpret_cast<const f2*>(pw);       // head[i][c][m]
    for (int i = t; i < NMODE * SW; i += INVM_T) {
      const int m = i % NMODE, ch = i / NMODE;
      f2 s = {0.f, 0.f};
#pragma unroll
      for (int c = 0; c < OUT; ++c) {
        const f2 a = go[c * NMODE + m], w = wh[(ch * OUT + c) * NMODE + m];
        s.x = fmaf(a.x, w.x, fmaf(a.y, w.y, s.x));
        s.y = fmaf(a.y, w.x, fmaf(-a.x, w.y, s.y));
      }
      gsm[m][ch] = s;
    }
  }
  // all loads go out before the first is waited for (arrays past their end read
  // the last entry again); G's, which the block waits for first, lead (one patch
  // in FP32: 8.7 us, 11.0 with each staging loop waiting by itself)
  typedef float float4v __attribute__((ext_vector_type(4)));
  constexpr int NG = SNM * SW / 2, NGQ = (NG + INVM_T - 1) / INVM_T;
  constexpr int NYQ = (SN * KY + INVM_T - 1) / INVM_T;
  float4v gv[NGQ];
  f2 yv[NYQ];
  if constexpr (MODE != INV_HEAD) {
    const float4v* gb = reinterpret_cast<const float4v*>(G + (long long)b * SNM * SW);
#pragma unroll
    for (int k = 0; k < NGQ; ++k) gv[k] = gb[min(t + INVM_T * k, NG - 1)];
  }
#pragma unroll
  for (int k = 0; k < NYQ; ++k) yv[k] = iy[min(t + INVM_T * k, SN * KY - 1)];
  // fixed operands: A = pw^T (row o = li, k = i), B = row-transform twiddles
  // (k' < KX: Re ix[k'][x], else -Im ix[k' - KX][x]; column x = li)
  float pwa[SW / 2], ixb[KX];
  if constexpr (MODE != INV_HEAD)
#pragma unroll
    for (int s = 0; s < SW / 2; ++s)
      pwa[s] = op<BF16>(MODE == INV_LAYER ? pw[(2 * s + lh) * SW + li] : pw[li * SW + 2 * s + lh]);
#pragma unroll
  for (int s = 0; s < KX; ++s) {
    const int k = 2 * s + lh;
    ixb[s] = k < KX ? op<BF16>(ix[k * SN + li]).x : -op<BF16>(ix[(k - KX) * SN + li]).y;
  }
  const float* hb = h + (long long)b * SW * SN * SN;
  // this wave's pixels of its row: B operand of the pointwise part (k = i);
  // the next row's are loaded as soon as the current ones are consumed
  float hv[SW / 2];
  if constexpr (MODE != INV_HEAD)
#pragma unroll
    for (int s = 0; s < SW / 2; ++s)
      hv[s] = ld<NT>(&hb[((2 * s + lh) * SN + inv_row(g0, wave)) * SN + li]);
  if constexpr (MODE != INV_HEAD)
#pragma unroll
    for (int k = 0; k < NGQ; ++k) {
      f2* dst = &gsm[0][0] + 2 * min(t + INVM_T * k, NG - 1);
      dst[0] = op<BF16>(f2{gv[k].x, gv[k].y});
      dst[1] = op<BF16>(f2{gv[k].z, gv[k].w});
    }
#pragma unroll
  for (int k = 0; k < NYQ; ++k) iys[min(t + INVM_T * k, SN * KY - 1)] = op<BF16>(yv[k]);
  for (int yc = g0; yc < g0 + groups; ++yc) {
    const int y = inv_row(yc, wave);
    __syncthreads();  // G staged (first group) / the previous group's gy consumed
    // column transform of the group's 4 row pairs: items (pair, kx, o), o fastest
    for (int it = t; it < 4 * KX * SW; it += INVM_T) {
      const int o = it % SW, kx = (it / SW) % KX, pr = it / (SW * KX);
      const int ya = inv_row(yc, pr), yb = inv_row(yc, pr + 4);
      float ra = 0.f, ia = 0.f, rb = 0.f, ib = 0.f;
      if (ya == 0) {  // rows 0 and 16
#pragma unroll 4
        for (int ky = 0; ky < KY; ++ky) {
          const f2 v = gsm[ky * KX + kx][o], a = iys[ya * KY + ky], c = iys[yb * KY + ky];
          ra = fmaf(a.x, v.x, fmaf(-a.y, v.y, ra));
          ia = fmaf(a.x, v.y, fmaf(a.y, v.x, ia));
          rb = fmaf(c.x, v.x, fmaf(-c.y, v.y, rb));
          ib = fmaf(c.x, v.y, fmaf(c.y, v.x, ib));
        }
      } else {
        float ar = 0.f, ai = 0.f, br = 0.f, bi = 0.f;
#pragma unroll
        for (int ky = 0; ky < KY; ++ky) {
          const f2 v = gsm[ky * KX + kx][o], a = iys[ya * KY + ky];
          ar = fmaf(a.x, v.x, ar);
          ai = fmaf(a.x, v.y, ai);
          br = fmaf(a.y, v.y, br);
          bi = fmaf(a.y, v.x, bi);
        }
        ra = ar - br;
        ia = ai + bi;
        rb = ar + br;
        ib = ai - bi;
      }
      gyl[pr][o][kx] = op<BF16>(ra);
      gyl[pr][o][KX + kx] = op<BF16>(ia);
      gyl[pr + 4][o][kx] = op<BF16>(rb);
      gyl[pr + 4][o][KX + kx] = op<BF16>(ib);
    }
    __syncthreads();
    floatx16 acc = {0};
    if constexpr (MODE != INV_HEAD) {
#pragma unroll
      for (int s = 0; s < SW / 2; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pwa[s], op<BF16>(hv[s]), acc, 0, 0, 0);
      if (yc + 1 < g0 + groups)  // rounded (BF16) where used, so the loads stay in flight
#pragma unroll
        for (int s = 0; s < SW / 2; ++s)
          hv[s] = ld<NT>(&hb[((2 * s + lh) * SN + inv_row(yc + 1, wave)) * SN + li]);
    }
#pragma unroll
    for (int s = 0; s < KX; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(gyl[wave][li][2 * s + lh], ixb[s], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int o = 8 * (r / 4) + 4 * lh + (r % 4);
      const long long off = (((long long)b * SW + o) * SN + y) * SN + li;
      if constexpr (MODE == INV_LAYER) {
        const float z = acc[r] + pb[o];
        if (z_out) z_out[off] = z;
        if (apply_gelu) st<NT>(&h_out[off], gelu_fwd_f(z));
        else if (h_out != z_out) st<NT>(&h_out[off], z);
      } else if (MODE == INV_ADJOINT && zp) {
        h_out[off] = acc[r] * gelu_grad_f(zp[off]);
      } else {
        h_out[off] = acc[r];
      }
    }
  }
}

// The head's mixing, 3 outputs: out[b][o][m] = sum_i A[b][i][m] W[i][o][m].
// One thread per (patch, mode), modes fastest: every channel's spectra of a
// patch are read as 64 consecutive modes per wave, the weights (small, cached)
// likewise, and each spectral value serves the NO outputs of a thread: all three,
// or one (blockIdx.z) where that leaves less than two blocks per CU.
template <bool BF16, int NO>
__global__ void __launch_bounds__(256) mode_mix_head(const f2* __restrict__ A,
                                                     const f2* __restrict__ Wt, int nmode, int B,
                                                     f2* __restrict__ out) {
  constexpr int O = 3;
  const int o0 = blockIdx.z * NO;
  const int m = blockIdx.x * 64 + (threadIdx.x & 63);
  const int b = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (m >= nmode || b >= B) return;
  const f2* a = A + (long long)b * SW * nmode + m;
  const f2* w = Wt + m;
  f2 acc[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o) acc[o] = f2{0.f, 0.f};
#pragma unroll 8
  for (int i = 0; i < SW; ++i) {
    const f2 v = op<BF16>(a[(long long)i * nmode]);
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      const f2 c = op<BF16>(w[(i * O + o0 + o) * nmode]);
      acc[o].x = fmaf(v.x, c.x, fmaf(-v.y, c.y, acc[o].x));
      acc[o].y = fmaf(v.x, c.y, fmaf(v.y, c.x, acc[o].y));
    }
  }
#pragma unroll
  for (int o = 0; o < NO; ++o) out[((long long)b * O + o0 + o) * nmode + m] = acc[o];
}

// Per-mode channel mixing of a Fourier layer on the matrix cores:
//   out[b][m][o] = sum_i A[m][b][i] Wm[m][i][o]   (complex, i, o < 32)
// with the spectra and the weights mode-major, as one real contraction over
// k = (part, i), K = 64, per mode:
//   Re(b, o) = sum_i Ar Wr - Ai Wi,   Im(b, o) = sum_i Ar Wi + Ai Wr,
// into two 32 x 32 FP32 accumulators (patches x outputs). Block = 32 patches x
// MM_G modes, one wave per mode. A mode's 32 x 32 tile of spectra is one
// contiguous 8 KB run, staged in LDS (rows padded); each lane reads its
// sixteen weights W[2s + half][lane] straight from memory (32 consecutive
// outputs per half-wave) and uses them for both halves of K; each half-wave
// writes the 32 outputs of one (patch, mode), one 256-byte run. With BF16 the operands are
// rounded to bf16 as they are read (their products are exact in FP32).
// All loads go out together, 16 bytes each for the spectra, and a lane reads both
// parts of a value at once: 4096 patches in FP32 (321 MB) 77 us, 64 in bf16
// products 6.2, one 4.9; with the weights read after the spectra were staged, by
// 8 bytes, 119, 12.4 and 6.7.
// ADJ is the adjoint, out[b][m][i] = sum_o A[m][b][o] conj(Wm[m][i][o]): a lane
// then takes channels o = 16 half + s in product s, so that its sixteen
// weights are one 128-byte run of its row i of Wm.
constexpr int MM_G = 4;
template <bool BF16, bool ADJ>
__global__ void __launch_bounds__(256) mode_mix_mm(const f2* __restrict__ A,
                                                   const f2* __restrict__ Wm, int nmode, int B,
                                                   f2* __restrict__ out) {
  __shared__ f2 as[MM_G][32][SW + 1];  // [mode][patch][i]
  typedef float float4v __attribute__((ext_vector_type(4)));
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, li = lane & 31, lh = lane >> 5;
  const int b0 = blockIdx.x * 32, m0 = blockIdx.y * MM_G;
  const int m = m0 + wave;
  // the weights' loads go out with the spectra's (a wave past the last mode
  // reads the last one's)
  const f2* wm = Wm + (long long)min(m, nmode - 1) * SW * SW;
  f2 wv[SW / 2];
#pragma unroll
  for (int s = 0; s < SW / 2; ++s)
    wv[s] = ADJ ? wm[li * SW + 16 * lh + s] : wm[(2 * s + lh) * SW + li];
  constexpr int NQ = MM_G * 32 * SW / 2 / 256;  // pairs of spectra per thread
  float4v av[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const int q = t + 256 * k, mm = q / (16 * SW), bb = (q / 16) % 32, i = 2 * (q % 16);
    const bool on = m0 + mm < nmode && b0 + bb < B;
    const long long at = on ? ((long long)(m0 + mm) * B + b0 + bb) * SW + i : 0;
    av[k] = *reinterpret_cast<const float4v*>(A + at);
    if (!on) av[k] = float4v{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const int q = t + 256 * k, mm = q / (16 * SW), bb = (q / 16) % 32, i = 2 * (q % 16);
    as[mm][bb][i] = op<BF16>(f2{av[k].x, av[k].y});
    as[mm][bb][i + 1] = op<BF16>(f2{av[k].z, av[k].w});
  }
  __syncthreads();
  if (m >= nmode) return;  // no barrier follows
#pragma unroll
  for (int s = 0; s < SW / 2; ++s) wv[s] = op<BF16>(ADJ ? f2{wv[s].x, -wv[s].y} : wv[s]);
  f2 a[SW / 2];
#pragma unroll
  for (int s = 0; s < SW / 2; ++s) a[s] = as[wave][li][ADJ ? 16 * lh + s : 2 * s + lh];
  floatx16 cre = {0}, cim = {0};
#pragma unroll
  for (int s = 0; s < SW / 2; ++s) {  // real parts of A
    cre = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s].x, wv[s].x, cre, 0, 0, 0);
    cim = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s].x, wv[s].y, cim, 0, 0, 0);
  }
#pragma unroll
  for (int s = 0; s < SW / 2; ++s) {  // imaginary parts of A
    cre = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s].y, -wv[s].y, cre, 0, 0, 0);
    cim = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s].y, wv[s].x, cim, 0, 0, 0);
  }
  f2* dst = out + ((long long)b0 * nmode + m) * SW + li;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int bb = 8 * (r / 4) + 4 * lh + (r % 4);
    if (b0 + bb < B) dst[(long long)bb * nmode * SW] = f2{cre[r], cim[r]};
  }
}

// Forward half of a layer and its mixing in one launch, for FP32 inference of few
// patches: G[b][m][o] = sum_i H[m][b][i] Wm[m][i][o] of the modes m of one kx.
// Grid (9, B), 576 threads: the block transforms all 1024 rows of the patch for
// its kx, then a thread per (ky, channel) the columns and a thread per (ky,
// output) the mixing, whose weights are loaded first of all. Each launch of a
// small batch costs its latency, and every block reads the whole patch again, so
// this pays while the blocks have a CU each: one patch 7.6 us, 10.9 in two
// launches; a call with 28 patches 99 us, 105.
//
// Every sum has the terms and the order of fused_dft_fwd and mode_mix_mm (whose
// FP32 products add their two K slots one after the other), so that a patch's
// result has the same bits in every batch, and as in the training forward pass.
constexpr int FM_T = 18 * 32;
__global__ void __launch_bounds__(FM_T) fwd_mix(const float* __restrict__ h,
                                                const f2* __restrict__ fy,
                                                const f2* __restrict__ fx,
                                                const f2* __restrict__ Wm,
                                                f2* __restrict__ G) {
  constexpr int HS = SN + 1, RS = SN + 4;  // row strides against bank conflicts
  __shared__ f2 hx[SW * HS], fys[SKY * HS], Hs[SKY * HS];
  __shared__ __attribute__((aligned(16))) float rows[8][SN * RS];
  const int t = threadIdx.x, kx = blockIdx.x, ch = t & 31, ky = t >> 5;
  const long long b = blockIdx.y;
  // Rows: eight lanes read a row of 128 bytes, a wave (the ninth has none) eight
  // rows per load and sixteen such groups: the 32 rows of four channels.
  constexpr int NR = 16;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, part = lane & 7;
  typedef float float4v __attribute__((ext_vector_type(4)));
  float4v rv[NR];
  if (wave < 8) {
    const float4v* src = reinterpret_cast<const float4v*>(
        h + (b * SW * SN + wave * NR * 8 + (lane >> 3)) * SN + 4 * part);
#pragma unroll
    for (int k = 0; k < NR; ++k) rv[k] = src[k * 8 * SN / 4];
  }
  const f2 yv = fy[min(t, SKY * SN - 1)];  // past the end: the last entry again
  const int m = min(ky, SKY - 1) * SKX + kx;
  f2 wv[SW];
  auto weights = [&](int i0) {  // half of them: with all from the start registers would spill
#pragma unroll
    for (int i = 0; i < SW / 2; ++i) wv[i0 + i] = Wm[((long long)m * SW + i0 + i) * SW + ch];
  };
  weights(0);
  if (t < SKY * SN) fys[(t / SN) * HS + t % SN] = yv;
  if (wave < 8) {
    // Through LDS a lane gets a whole row, the upper half-wave the same rows for
    // the imaginary part: with the twiddles of x and 32 - x conjugate, Re takes
    // row[x] + row[32 - x] and Im the difference.
    const int y = lane & 31;
    const bool imag = lane >= 32;
    const float sign = imag ? -1.f : 1.f;
    float w[SN / 2 + 1];
#pragma unroll
    for (int x = 0; x <= SN / 2; ++x) {
      const f2 v = fx[x * SKX + kx];  // wave-uniform
      w[x] = imag ? v.y : v.x;
    }
    float* stage = rows[wave];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c == 2) weights(SW / 2);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<float4v*>(stage + (8 * k + (lane >> 3)) * RS + 4 * part) = rv[4 * c + k];
      wave_sync();
      float row[SN];
#pragma unroll
      for (int q = 0; q < SN / 4; ++q) {
        const float4v v = *reinterpret_cast<const float4v*>(stage + y * RS + 4 * q);
        row[4 * q] = v.x;
        row[4 * q + 1] = v.y;
        row[4 * q + 2] = v.z;
        row[4 * q + 3] = v.w;
      }
      float s = fmaf(row[0], w[0], row[SN / 2] * w[SN / 2]);
#pragma unroll
      for (int x = 1; x < SN / 2; ++x) s = fmaf(fmaf(sign, row[SN - x], row[x]), w[x], s);
      reinterpret_cast<float*>(hx + (wave * 4 + c) * HS + y)[imag] = s;
      wave_sync();  // the rows are read before the next are staged
    }
  } else {
    weights(SW / 2);
  }
  __syncthreads();
  if (ky < SKY) {  // columns, rows yy and 32 - yy together
    const f2 *hc = hx + ch * HS, *a = fys + ky * HS;
    float re = 0.f, im = 0.f;
#pragma unroll
    for (int yy = 0; yy <= SN / 2; yy += SN / 2) {
      re = fmaf(a[yy].x, hc[yy].x, fmaf(-a[yy].y, hc[yy].y, re));
      im = fmaf(a[yy].x, hc[yy].y, fmaf(a[yy].y, hc[yy].x, im));
    }
#pragma unroll
    for (int yy = 1; yy < SN / 2; ++yy) {
      const f2 va = hc[yy], vb = hc[SN - yy], w = a[yy];
      re = fmaf(w.x, va.x + vb.x, fmaf(-w.y, va.y - vb.y, re));
      im = fmaf(w.x, va.y + vb.y, fmaf(w.y, va.x - vb.x, im));
    }
    Hs[ky * HS + ch] = f2{re, im};
  }
  __syncthreads();
  if (ky < SKY) {
    const f2* hs = Hs + ky * HS;
    f2 g = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < SW; ++i) {  // real parts of H
      g.x = fmaf(hs[i].x, wv[i].x, g.x);
      g.y = fmaf(hs[i].x, wv[i].y, g.y);
    }
#pragma unroll
    for (int i = 0; i < SW; ++i) {  // imaginary parts
      g.x = fmaf(hs[i].y, -wv[i].y, g.x);
      g.y = fmaf(hs[i].y, wv[i].x, g.y);
    }
    G[(b * SNM + m) * SW + ch] = g;
  }
}

// Mode-major copy of the layers' spectral weights: Wm[k][m][i][o] from
// W_k[i][o][m] (layer k at W + k * layer_stride complex values). A block takes
// one (i, k): 32 x nmode values that are one run of W, turned in LDS and
// written as nmode runs of 256 bytes. Grid (32, layers).
__global__ void __launch_bounds__(512) spec_mode_major(const f2* __restrict__ W,
                                                       long long layer_stride,
                                                       f2* __restrict__ Wm) {
  __shared__ f2 tile[SNM][SW + 1];
  const int t = threadIdx.x, i = blockIdx.x, k = blockIdx.y;
  const f2* src = W + k * layer_stride + (long long)i * SW * SNM;
  for (int q = t; q < SW * SNM; q += 512) tile[q % SNM][q / SNM] = src[q];
  __syncthreads();
  f2* dst = Wm + ((long long)k * SNM * SW + i) * SW;
  for (int q = t; q < SW * SNM; q += 512)
    dst[(long long)(q / SW) * SW * SW + q % SW] = tile[q / SW][q % SW];
}

// The lift: h[b][o][p] = sum_c lw[c][o] x[b][c][p] + lb[o], 16 input and 32
// output channels, 2 pixels per thread. Grid (B, P, Q): a block takes 1024 / P
// pixels and 32 / Q outputs; small batches are split to reach more CUs (one
// patch: 6.5 us in one block, 4.5 in eight).
template <bool BF16>
__global__ void __launch_bounds__(512) lift_kernel(const float* __restrict__ x,
                                                   const float* __restrict__ lw,
                                                   const float* __restrict__ lb,
                                                   float* __restrict__ h) {
  constexpr int CI = 16;
  __shared__ float lws[CI * SW], lbs[SW];
  const int b = blockIdx.x, t = blockIdx.y * blockDim.x + threadIdx.x;
  const int no = SW / gridDim.z, o0 = blockIdx.z * no;
  for (int i = threadIdx.x; i < CI * SW; i += blockDim.x) lws[i] = op<BF16>(lw[i]);
  if (threadIdx.x < SW) lbs[threadIdx.x] = lb[threadIdx.x];
  float xr[CI][2];
  const float* xb = x + (long long)b * CI * SN * SN;
#pragma unroll
  for (int c = 0; c < CI; ++c) {
    const float2 v = *reinterpret_cast<const float2*>(xb + c * SN * SN + 2 * t);
    xr[c][0] = op<BF16>(v.x);
    xr[c][1] = op<BF16>(v.y);
  }
  __syncthreads();
  float* hb = h + (long long)b * SW * SN * SN + 2 * t;
#pragma unroll 4
  for (int o = o0; o < o0 + no; ++o) {
    float a0 = lbs[o], a1 = lbs[o];
#pragma unroll
    for (int c = 0; c < CI; ++c) {
      const float w = lws[c * SW + o];
      a0 = fmaf(w, xr[c][0], a0);
      a1 = fmaf(w, xr[c][1], a1);
    }
    *reinterpret_cast<float2*>(hb + o * SN * SN) = make_float2(a0, a1);
  }
}

// complex64 index patches [B][8][32][32] -> channels [B][16][32][32], one
// (patch, layer) per block and four pixels per thread; VEC: in 16-byte accesses
// (both arrays aligned), NT: non-temporal. Bound by memory: 537 MB in 88 us,
// 117 with one pixel per thread.
template <bool VEC, bool NT>
__global__ void __launch_bounds__(256) encode(const float* n, float* x) {
  typedef float float4v __attribute__((ext_vector_type(4)));
  constexpr int P = SN * SN;
  const long long bl = blockIdx.x;  // b * 8 + l
  const int p = 4 * threadIdx.x;
  const float* src = n + (bl * P + p) * 2;
  float* re = x + bl * 2 * P + p;  // channel 2 l of patch b, then 2 l + 1
  float* im = re + P;
  if constexpr (VEC) {
    const float4v* s4 = reinterpret_cast<const float4v*>(src);
    const float4v a = NT ? __builtin_nontemporal_load(s4) : s4[0];
    const float4v c = NT ? __builtin_nontemporal_load(s4 + 1) : s4[1];
    const float4v r = {(a.x - 1.45f) / 0.15f, (a.z - 1.45f) / 0.15f, (c.x - 1.45f) / 0.15f,
                       (c.z - 1.45f) / 0.15f};
    const float4v i = {a.y / 0.05f, a.w / 0.05f, c.y / 0.05f, c.w / 0.05f};
    if constexpr (NT) {
      __builtin_nontemporal_store(r, reinterpret_cast<float4v*>(re));
      __builtin_nontemporal_store(i, reinterpret_cast<float4v*>(im));
    } else {
      *reinterpret_cast<float4v*>(re) = r;
      *reinterpret_cast<float4v*>(im) = i;
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      re[k] = (src[2 * k] - 1.45f) / 0.15f;
      im[k] = src[2 * k + 1] / 0.05f;
    }
  }
}

inline unsigned blocks(long long n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t sur_adam(float* p, const float* g, float* m, float* v, long long n, float lr, int t,
                    hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  adam<<<blocks(n), 256, 0, s>>>(p, g, m, v, n, lr, b1, b2, 1e-8f, c1, c2);
  return hipGetLastError();
}
hipError_t sur_fused_dft_fwd(const float* h, const float* fy, const float* fx, float* H, int B,
                            bool head, bool bf16, hipStream_t s) {
  dim3 grid(SW / 8, B);
  auto go = [&](auto kern, int T) {
    kern<<<grid, 256 * T, 0, s>>>(h, reinterpret_cast<const f2*>(fy),
                                  reinterpret_cast<const f2*>(fx), reinterpret_cast<f2*>(H));
  };
  auto pick = [&](auto rounded) {
    constexpr bool R = decltype(rounded)::value;
    if (head) {  // the head's centred 15 x 15 band, [b][i][mode]
      if (B <= 64) go(fused_dft_fwd<R, 15, 15, false, 2>, 2);
      else go(fused_dft_fwd<R, 15, 15, false, 1>, 1);
    } else {  // a Fourier layer's 17 x 9 half plane, [mode][b][i]
      if (B <= 64) go(fused_dft_fwd<R, SKY, SKX, true, 2>, 2);
      else go(fused_dft_fwd<R, SKY, SKX, true, 1>, 1);
    }
  };
  if (bf16) pick(std::true_type{});
  else pick(std::false_type{});
  return hipGetLastError();
}
// Row-group splits of the inverse half: as many as keep the launch within two
// blocks per CU (what its LDS allows), since every split stages G again.
static int inv_splits(int B) { return B <= 128 ? 4 : B <= 256 ? 2 : 1; }

hipError_t sur_fused_dft_inv(const float* G, const float* h, const float* iy, const float* ix,
                             const float* pw, const float* pb, float* z_out, float* h_out,
                             bool gelu, int B, bool bf16, hipStream_t s) {
  auto go = [&](auto kern) {
    kern<<<dim3(B, inv_splits(B)), INVM_T, 0, s>>>(
        reinterpret_cast<const f2*>(G), h, reinterpret_cast<const f2*>(iy),
        reinterpret_cast<const f2*>(ix), pw, pb, z_out, h_out, gelu ? 1 : 0, nullptr);
  };
  if (bf16) go(fused_dft_inv_mfma<true, INV_LAYER>);
  else if (sur_past_cache(2 * B)) go(fused_dft_inv_mfma<false, INV_LAYER, true>);
  else go(fused_dft_inv_mfma<false, INV_LAYER>);
  return hipGetLastError();
}
hipError_t sur_fused_dft_adjoint(const float* gH, const float* gz, const float* fyh,
                                 const float* fxh, const float* pw, const float* zp, float* out,
                                 int B, hipStream_t s) {
  fused_dft_inv_mfma<false, INV_ADJOINT><<<dim3(B, inv_splits(B)), INVM_T, 0, s>>>(
      reinterpret_cast<const f2*>(gH), gz, reinterpret_cast<const f2*>(fyh),
      reinterpret_cast<const f2*>(fxh), pw, nullptr, nullptr, out, 0, zp);
  return hipGetLastError();
}
hipError_t sur_head_adjoint(const float* gout, const float* head, const float* hyh,
                            const float* hxh, float* out, int B, hipStream_t s) {
  fused_dft_inv_mfma<false, INV_HEAD><<<dim3(B, inv_splits(B)), INVM_T, 0, s>>>(
      reinterpret_cast<const f2*>(gout), nullptr, reinterpret_cast<const f2*>(hyh),
      reinterpret_cast<const f2*>(hxh), head, nullptr, nullptr, out, 0, nullptr);
  return hipGetLastError();
}
hipError_t sur_mode_mix(const float* A, const float* W, int nmode, int B, int O, float* out,
                        bool bf16, hipStream_t s) {
  const f2* a = reinterpret_cast<const f2*>(A);
  const f2* w = reinterpret_cast<const f2*>(W);
  f2* o = reinterpret_cast<f2*>(out);
  if (O == 3) {
    dim3 grid((nmode + 63) / 64, (B + 3) / 4);
    auto go = [&](auto kern) { kern<<<grid, 256, 0, s>>>(a, w, nmode, B, o); };
    if (grid.x * grid.y < 512) {
      grid.z = 3;
      if (bf16) go(mode_mix_head<true, 1>);
      else go(mode_mix_head<false, 1>);
    } else {
      if (bf16) go(mode_mix_head<true, 3>);
      else go(mode_mix_head<false, 3>);
    }
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
hipError_t sur_mode_mix_layer(const float* A, const float* Wm, int nmode, int B, float* out,
                              bool bf16, hipStream_t s) {
  dim3 grid((B + 31) / 32, (nmode + MM_G - 1) / MM_G);
  const f2* a = reinterpret_cast<const f2*>(A);
  const f2* w = reinterpret_cast<const f2*>(Wm);
  f2* o = reinterpret_cast<f2*>(out);
  if (bf16) mode_mix_mm<true, false><<<grid, 256, 0, s>>>(a, w, nmode, B, o);
  else mode_mix_mm<false, false><<<grid, 256, 0, s>>>(a, w, nmode, B, o);
  return hipGetLastError();
}
hipError_t sur_fwd_mix(const float* h, const float* fy, const float* fx, const float* Wm, int B,
                       float* G, hipStream_t s) {
  fwd_mix<<<dim3(SKX, B), FM_T, 0, s>>>(h, reinterpret_cast<const f2*>(fy),
                                        reinterpret_cast<const f2*>(fx),
                                        reinterpret_cast<const f2*>(Wm),
                                        reinterpret_cast<f2*>(G));
  return hipGetLastError();
}
hipError_t sur_mode_mix_adjoint(const float* A, const float* Wm, int nmode, int B, float* out,
                                hipStream_t s) {
  dim3 grid((B + 31) / 32, (nmode + MM_G - 1) / MM_G);
  mode_mix_mm<false, true><<<grid, 256, 0, s>>>(reinterpret_cast<const f2*>(A),
                                                reinterpret_cast<const f2*>(Wm), nmode, B,
                                                reinterpret_cast<f2*>(out));
  return hipGetLastError();
}
hipError_t sur_spec_mode_major(const float* W, long long layer_stride_floats, int nmode,
                               int layers, float* Wm, hipStream_t s) {
  if (layer_stride_floats % 2 != 0 || nmode != SNM) return hipErrorInvalidValue;
  spec_mode_major<<<dim3(SW, layers), 512, 0, s>>>(reinterpret_cast<const f2*>(W),
                                                   layer_stride_floats / 2,
                                                   reinterpret_cast<f2*>(Wm));
  return hipGetLastError();
}
hipError_t sur_lift(const float* x, const float* lw, const float* lb, float* h, int B, bool bf16,
                    hipStream_t s) {
  const int P = B <= 64 ? 2 : 1, Q = B <= 64 ? 4 : 1;
  const dim3 grid(B, P, Q);
  auto go = [&](auto kern) { kern<<<grid, 512 / P, 0, s>>>(x, lw, lb, h); };
  if (bf16) go(lift_kernel<true>);
  else go(lift_kernel<false>);
  return hipGetLastError();
}
hipError_t sur_encode(const float* n, float* x, int B, hipStream_t s) {
  const bool vec = (reinterpret_cast<uintptr_t>(n) | reinterpret_cast<uintptr_t>(x)) % 16 == 0;
  auto go = [&](auto kern) { kern<<<8 * B, 256, 0, s>>>(n, x); };
  if (!vec) go(encode<false, false>);
  else if (sur_past_cache(B)) go(encode<true, true>);
  else go(encode<true, false>);
  return hipGetLastError();
}

}  // namespace scw
