// Backward kernels of the surrogate: the loss, the weight gradients, and the
// adjoint of the network in bf16 products. (The FP32 adjoint runs the forward
// kernels of kernels_surrogate.hip with adjoint tables and weights.)
//
// A layer's adjoint is four launches and its weight gradients three, each
// reading its inputs once. With one strided GEMM launch per linear step (eight
// per layer, intermediates of 2-9 MB per 64 patches between them, tiles padded
// from 9 or 17 columns to 64) and one block per channel for the biases, a loss
// and gradient took 2.27 ms in bf16 products at 64 patches and 4.93 ms in FP32
// at 256, against 0.65 and 1.10 ms as here.
//
// The bf16 adjoint rounds both operands of every product to bf16 (nearest
// even) and sums in FP32 on v_mfma_f32_32x32x16_bf16 over K in its natural
// order, 16 at a time; a complex product takes, per K step,
//   Re += Re A Re B,  Im += Re A Im B,  Re += (-Im A) Im B,  Im += Im A Re B.
// That order is part of the results: an intermediate that differs in its last
// FP32 bit can round to another bf16 operand, and within a few layers such
// flips reach 1e-3 of the gradient. MFMA lane layout (one wave, 32 x 32 x 16):
// lane l holds A[l % 32][8 (l / 32) + 0..7] and B[8 (l / 32) + 0..7][l % 32];
// accumulator r of lane l is D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32].
#include <hip/hip_runtime.h>

#include <algorithm>

#include "scw_internal.h"
#include "surrogate_device.h"

namespace scw {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int HN = 15, HM = HN * HN, OUT = 3;  // head band, outputs

__device__ __forceinline__ floatx16 mm16(bf16x8 a, bf16x8 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 neg8(bf16x8 a) {  // every bf16 sign flipped
  return __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, a) ^ 0x80008000u);
}
__device__ __forceinline__ int drow(int r, int lh) { return 8 * (r / 4) + 4 * lh + (r % 4); }

// ---------------------------------------------------------------- loss
// part[0][c] = sum_j |out - tgt|^2 and part[1][c] = sum_j |tgt|^2 over the
// complex entries c + 256 j, for the 256 chains c; sums[0], sums[1] are their
// totals by a binary tree. Each chain is summed in the order of j, so it is a
// serial chain of FP32 adds: a block takes 16 chains (128-byte runs) and forms
// 64 of their terms at a time in parallel, which leaves the chain only LDS
// reads and adds. Grid 16. (One block for all chains, with the loads inside
// the chain: 283 us for 172,800 entries, 47 us for 43,200.)
constexpr int LC = 16, LJ = 64;
__global__ void __launch_bounds__(256) loss_chains(const float* __restrict__ out,
                                                   const float* __restrict__ tgt, long long n,
                                                   float* __restrict__ part) {
  __shared__ float ta[LJ][LC], tb[LJ][LC];
  const int t = threadIdx.x, cc = t % LC, jj = t / LC;  // 16 chains x 16 rows
  const long long c0 = blockIdx.x * LC + cc;
  const f2* o2 = reinterpret_cast<const f2*>(out);
  const f2* t2 = reinterpret_cast<const f2*>(tgt);
  const long long nj = (n + 255) / 256;
  float s = 0.f;
  for (long long j0 = 0; j0 < nj; j0 += LJ) {
    f2 o[LJ / 16], g[LJ / 16];
#pragma unroll
    for (int q = 0; q < LJ / 16; ++q) {
      const long long i = c0 + 256 * (j0 + jj + 16 * q);
      o[q] = g[q] = f2{0.f, 0.f};
      if (i < n) {
        o[q] = o2[i];
        g[q] = t2[i];
      }
    }
    __syncthreads();  // the previous terms have been added
#pragma unroll
    for (int q = 0; q < LJ / 16; ++q) {
      const float dx = o[q].x - g[q].x, dy = o[q].y - g[q].y;
      ta[jj + 16 * q][cc] = dx * dx + dy * dy;
      tb[jj + 16 * q][cc] = g[q].x * g[q].x + g[q].y * g[q].y;
    }
    __syncthreads();
    if (t < 2 * LC) {  // entries past the end add zero
      const float (*tt)[LC] = t < LC ? ta : tb;
#pragma unroll 16
      for (int j = 0; j < LJ; ++j) s += tt[j][cc];
    }
  }
  if (t < 2 * LC) part[(t / LC) * 256 + c0] = s;
}

// The tree over the chains (every block forms it again), the totals by block
// 0, and g = 2 (out - tgt) / sums[1].
__global__ void __launch_bounds__(256) loss_grad(const float* __restrict__ out,
                                                 const float* __restrict__ tgt,
                                                 const float* __restrict__ part,
                                                 float* __restrict__ sums, float* __restrict__ g,
                                                 long long n2) {
  __shared__ float r0[256], r1[256];
  r0[threadIdx.x] = part[threadIdx.x];
  r1[threadIdx.x] = part[256 + threadIdx.x];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      r0[threadIdx.x] += r0[threadIdx.x + w];
      r1[threadIdx.x] += r1[threadIdx.x + w];
    }
    __syncthreads();
  }
  const float den = r1[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sums[0] = r0[0];
    sums[1] = den;
  }
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < n2) g[i] = 2.f * (out[i] - tgt[i]) / den;
}

// ---------------------------------------------------------------- weight gradients
// out[e] = sum_p part[p][e], e < E, for every job: 32 entries x 8 slices of the
// parts per block, the jobs' blocks one after another (one launch for all of a
// gradient's sums: apart they took 6 x 3.9 us).
__global__ void __launch_bounds__(256) sum_parts(const SurSumJobs jobs) {
  __shared__ float red[8][33];
  int q = 0, blk = blockIdx.x;
  for (; blk >= (jobs.j[q].E + 31) / 32; ++q) blk -= (jobs.j[q].E + 31) / 32;
  const float* __restrict__ part = jobs.j[q].part;
  const int P = jobs.j[q].P, E = jobs.j[q].E;
  float* __restrict__ out = jobs.j[q].out;
  const int el = threadIdx.x & 31, sl = threadIdx.x >> 5;
  const int e = blk * 32 + el;
  float s = 0.f;
  if (e < E)
#pragma unroll 8
    for (int p = sl; p < P; p += 8) s += part[(long long)p * E + e];
  red[sl][el] = s;
  __syncthreads();
  if (sl == 0 && e < E) {
#pragma unroll
    for (int q = 1; q < 8; ++q) s += red[q][el];
    out[e] = s;
  }
}

// Pointwise weights and bias: part[blk][i][o] = sum h[b][i][p] gz[b][o][p] and
// part[blk][CI * 32 + o] = sum gz[b][o][p] over the block's units, a unit being
// a quarter (256 pixels) of a patch; wave w takes 64 of them. One pass over h
// and gz serves both gradients. A K step takes 8 (FP32: 4 products of K = 2)
// or 16 (bf16) consecutive pixels; a lane's are one or two 16-byte loads of
// its row. With CI = 16 the upper half of the tile is idle.
template <bool BF16, int CI>
__global__ void __launch_bounds__(256) pointwise_grad(const float* __restrict__ h,
                                                      const float* __restrict__ gz, int units,
                                                      float* __restrict__ part) {
  constexpr int NP = SN * SN, E = CI * SW + SW;
  __shared__ float red[3][16][64];
  __shared__ float bred[4][64];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, li = lane & 31, lh = lane >> 5;
  floatx16 acc = {0};
  float bias = 0.f;
  for (int u = blockIdx.x; u < units; u += gridDim.x) {
    const long long b = u >> 2;
    const int p0 = (u & 3) * 256 + wave * 64;
    const float* hr = h + (b * CI + (li & (CI - 1))) * NP + p0;
    const float* gr = gz + (b * SW + li) * NP + p0;
    if constexpr (BF16) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        bf16x8 a, g;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int o = 16 * s + 8 * lh + 4 * q;
          const float4 hv = *reinterpret_cast<const float4*>(hr + o);
          const float4 gv = *reinterpret_cast<const float4*>(gr + o);
          const float hh[4] = {hv.x, hv.y, hv.z, hv.w}, gg[4] = {gv.x, gv.y, gv.z, gv.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            a[4 * q + e] = (__bf16)hh[e];
            g[4 * q + e] = (__bf16)gg[e];
            bias += gg[e];
          }
        }
        acc = mm16(a, g, acc);
      }
    } else {
      float4 hv[8], gv[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        hv[s] = *reinterpret_cast<const float4*>(hr + 8 * s + 4 * lh);
        gv[s] = *reinterpret_cast<const float4*>(gr + 8 * s + 4 * lh);
      }
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(hv[s].x, gv[s].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(hv[s].y, gv[s].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(hv[s].z, gv[s].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(hv[s].w, gv[s].w, acc, 0, 0, 0);
        bias += (gv[s].x + gv[s].y) + (gv[s].z + gv[s].w);
      }
    }
  }
  if (wave > 0)
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave - 1][r][lane] = acc[r];
  bred[wave][lane] = bias;
  __syncthreads();
  float* dst = part + (long long)blockIdx.x * E;
  if (wave == 0) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = drow(r, lh);
      const float v = ((acc[r] + red[0][r][lane]) + red[1][r][lane]) + red[2][r][lane];
      if (i < CI) dst[i * SW + li] = v;
    }
    if (lane < SW) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) v += bred[w][lane] + bred[w][lane + 32];
      dst[CI * SW + lane] = v;
    }
  }
}

// Spectral weights of one layer, mode-major: gW[m][i][o] = sum_b
// conj(H[m][b][i]) gG[m][b][o]. One block per mode, its four waves taking
// every fourth K step (FP32: 2 patches, bf16: 16) of the sum over the batch;
// each half-wave's loads are 256-byte runs.
template <bool BF16>
__global__ void __launch_bounds__(256) spectral_grad(const f2* __restrict__ H,
                                                     const f2* __restrict__ gG, int B,
                                                     f2* __restrict__ gW) {
  __shared__ f2 red[3][16][64];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, li = lane & 31, lh = lane >> 5;
  const long long m = blockIdx.x;
  const f2* hm = H + m * B * SW + li;
  const f2* gm = gG + m * B * SW + li;
  floatx16 re = {0}, im = {0};
  if constexpr (BF16) {
    for (int b0 = 16 * wave; b0 < B; b0 += 64) {
      bf16x8 hr, hi, gr, gi;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int b = b0 + 8 * lh + j;
        const f2 hv = hm[(long long)min(b, B - 1) * SW], gv = gm[(long long)min(b, B - 1) * SW];
        hr[j] = (__bf16)(b < B ? hv.x : 0.f);
        hi[j] = (__bf16)(b < B ? hv.y : 0.f);
        gr[j] = (__bf16)gv.x;
        gi[j] = (__bf16)gv.y;
      }
      re = mm16(hr, gr, re);
      im = mm16(hr, gi, im);
      re = mm16(hi, gi, re);
      im = mm16(neg8(hi), gr, im);
    }
  } else {
#pragma unroll 4
    for (int b0 = 2 * wave; b0 < B; b0 += 8) {
      const int b = b0 + lh, bc = min(b, B - 1);
      f2 hv = hm[(long long)bc * SW];
      const f2 gv = gm[(long long)bc * SW];
      if (b >= B) hv = f2{0.f, 0.f};
      re = __builtin_amdgcn_mfma_f32_32x32x2f32(hv.x, gv.x, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f32_32x32x2f32(hv.x, gv.y, im, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f32_32x32x2f32(hv.y, gv.y, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f32_32x32x2f32(-hv.y, gv.x, im, 0, 0, 0);
    }
  }
  if (wave > 0)
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave - 1][r][lane] = f2{re[r], im[r]};
  __syncthreads();
  if (wave > 0) return;
  f2* dst = gW + m * SW * SW + li;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    f2 v = {re[r], im[r]};
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      v.x += red[w][r][lane].x;
      v.y += red[w][r][lane].y;
    }
    dst[drow(r, lh) * SW] = v;
  }
}

// The layers' mode-major spectral gradients back into the parameter order,
// G_k[i][o][m] (layer k at G + k * layer_stride): spec_mode_major's inverse.
// Grid (32, layers).
__global__ void __launch_bounds__(512) spec_from_mode_major(const f2* __restrict__ gW,
                                                            long long layer_stride,
                                                            f2* __restrict__ G) {
  __shared__ f2 tile[SNM][SW + 1];
  const int t = threadIdx.x, i = blockIdx.x, k = blockIdx.y;
  const f2* src = gW + ((long long)k * SNM * SW + i) * SW;
  for (int q = t; q < SW * SNM; q += 512)
    tile[q / SW][q % SW] = src[(long long)(q / SW) * SW * SW + q % SW];
  __syncthreads();
  f2* dst = G + k * layer_stride + (long long)i * SW * SNM;
  for (int q = t; q < SW * SNM; q += 512) dst[q] = tile[q % SNM][q / SNM];
}

// Head weights: part[slice][i][c][m] = sum_b conj(F[b][i][m]) gout[b][c][m] over
// the slice's patches. Lanes run over modes, waves over channels i.
// Grid (4, 8, slices).
template <bool BF16>
__global__ void __launch_bounds__(256) head_grad(const f2* __restrict__ F,
                                                 const f2* __restrict__ gout, int B,
                                                 f2* __restrict__ part) {
  const int m = blockIdx.x * 64 + (threadIdx.x & 63), i = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (m >= HM) return;
  f2 acc[OUT];
#pragma unroll
  for (int c = 0; c < OUT; ++c) acc[c] = f2{0.f, 0.f};
#pragma unroll 4
  for (int b = blockIdx.z; b < B; b += gridDim.z) {
    const f2 f = op<BF16>(F[((long long)b * SW + i) * HM + m]);
#pragma unroll
    for (int c = 0; c < OUT; ++c) {
      const f2 g = op<BF16>(gout[((long long)b * OUT + c) * HM + m]);
      acc[c].x = fmaf(f.x, g.x, fmaf(f.y, g.y, acc[c].x));
      acc[c].y = fmaf(f.x, g.y, fmaf(-f.y, g.x, acc[c].y));
    }
  }
#pragma unroll
  for (int c = 0; c < OUT; ++c)
    part[(((long long)blockIdx.z * SW + i) * OUT + c) * HM + m] = acc[c];
}

// ---------------------------------------------------------------- bf16 adjoint
// gF[b][m][i] = sum_c gout[b][c][m] conj(head[i][c][m]) on 32 patches x 8 modes
// per block, a wave per mode (neighbouring modes share the lines they gather).
__global__ void __launch_bounds__(512) head_mix_adjoint_bf16(const f2* __restrict__ gout,
                                                             const f2* __restrict__ head, int B,
                                                             f2* __restrict__ gF) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
  const int b0 = blockIdx.x * 32, m = blockIdx.y * 8 + wave;
  if (m >= HM) return;
  const int b = b0 + li;
  bf16x8 ar, ai, br, bi;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const bool on = lh == 0 && j < OUT;
    f2 a = {0.f, 0.f}, w = {0.f, 0.f};
    if (on && b < B) a = gout[((long long)b * OUT + j) * HM + m];
    if (on) w = head[(li * OUT + j) * HM + m];
    ar[j] = (__bf16)a.x;
    ai[j] = (__bf16)a.y;
    br[j] = (__bf16)w.x;
    bi[j] = (__bf16)-w.y;
  }
  floatx16 cre = {0}, cim = {0};
  cre = mm16(ar, br, cre);
  cim = mm16(ar, bi, cim);
  cre = mm16(neg8(ai), bi, cre);
  cim = mm16(ai, br, cim);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int bb = b0 + drow(r, lh);
    if (bb < B) gF[((long long)bb * HM + m) * SW + li] = f2{cre[r], cim[r]};
  }
}

// gH[b][m][i] = sum_o gG[m][b][o] conj(Wm[m][i][o]): 32 patches x 4 modes per
// block, a wave per mode; a lane's operands are 64-byte runs of its row.
__global__ void __launch_bounds__(256) mode_mix_adjoint_bf16(const f2* __restrict__ gG,
                                                             const f2* __restrict__ Wm, int B,
                                                             f2* __restrict__ gH) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
  const int b0 = blockIdx.x * 32, m = blockIdx.y * 4 + wave;
  if (m >= SNM) return;
  const f2* ga = gG + ((long long)m * B + min(b0 + li, B - 1)) * SW;  // past the batch: unused rows
  const f2* wb = Wm + ((long long)m * SW + li) * SW;
  floatx16 cre = {0}, cim = {0};
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    bf16x8 ar, ai, br, bi;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const f2 a = ga[16 * s + 8 * lh + j], w = wb[16 * s + 8 * lh + j];
      ar[j] = (__bf16)a.x;
      ai[j] = (__bf16)a.y;
      br[j] = (__bf16)w.x;
      bi[j] = (__bf16)-w.y;
    }
    cre = mm16(ar, br, cre);
    cim = mm16(ar, bi, cim);
    cre = mm16(neg8(ai), bi, cre);
    cim = mm16(ai, br, cim);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int bb = b0 + drow(r, lh);
    if (bb < B) gH[((long long)bb * SNM + m) * SW + li] = f2{cre[r], cim[r]};
  }
}

// gG[m][b][o] = sum_y conj(iy[y][ky]) sum_x gz[b][o][y][x] conj(ix[kx][x]), the
// adjoint of the inverse half's transforms; 32 / S channels of one patch per
// block of 8 waves, grid (B, S). Rows: a wave transforms its 4 / S channels,
// D[y][Re kx | Im kx] over x. The rounded results go to LDS along y, the K of the
// columns, D[ky][o] per kx.
constexpr int T2S = 40;  // LDS row: 32 y + 8 pad (bf16), 16-byte aligned
template <int S>
__global__ void __launch_bounds__(512) dft_adjoint_bf16(const float* __restrict__ gz,
                                                        const f2* __restrict__ iy,
                                                        const f2* __restrict__ ix, int B,
                                                        f2* __restrict__ gG) {
  constexpr int CH = SW / S;
  __shared__ __attribute__((aligned(16))) __bf16 t2[SKX][2][CH][T2S];
  const int c0 = blockIdx.y * CH;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
  const long long b = blockIdx.x;
  // the pixels' loads lead the tables'
  float4 gv[CH / 8][4];
#pragma unroll
  for (int q = 0; q < CH / 8; ++q) {
    const float* row = gz + ((b * SW + c0 + wave * (CH / 8) + q) * SN + li) * SN;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      gv[q][s] = *reinterpret_cast<const float4*>(row + 16 * (s / 2) + 8 * lh + 4 * (s % 2));
  }
  const int kxl = li % SKX;  // column li < 18 of the row transform: kx, Re or Im
  const bool imag = li >= SKX;
  bf16x8 bx[2], ar[2], ai[2];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = 16 * s + 8 * lh + j;
      const f2 w = ix[kxl * SN + k];
      bx[s][j] = (__bf16)(li < 2 * SKX ? (imag ? -w.y : w.x) : 0.f);
      const f2 v = iy[k * SKY + min(li, SKY - 1)];
      ar[s][j] = (__bf16)(li < SKY ? v.x : 0.f);
      ai[s][j] = (__bf16)(li < SKY ? -v.y : 0.f);
    }
#pragma unroll
  for (int q = 0; q < CH / 8; ++q) {
    const int o = wave * (CH / 8) + q;
    floatx16 d = {0};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const float4 v0 = gv[q][2 * s], v1 = gv[q][2 * s + 1];
      const bf16x8 a = {(__bf16)v0.x, (__bf16)v0.y, (__bf16)v0.z, (__bf16)v0.w,
                        (__bf16)v1.x, (__bf16)v1.y, (__bf16)v1.z, (__bf16)v1.w};
      d = mm16(a, bx[s], d);
    }
    if (li < 2 * SKX) {
      __bf16* dst = t2[kxl][imag ? 1 : 0][o];
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[drow(r, lh)] = (__bf16)d[r];
    }
  }
  __syncthreads();
  const int lc = li & (CH - 1);  // column li of the product; li >= CH repeats, unused
  for (int kx = wave; kx < SKX; kx += 8) {
    floatx16 cre = {0}, cim = {0};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const bf16x8 br = *reinterpret_cast<const bf16x8*>(&t2[kx][0][lc][16 * s + 8 * lh]);
      const bf16x8 bi = *reinterpret_cast<const bf16x8*>(&t2[kx][1][lc][16 * s + 8 * lh]);
      cre = mm16(ar[s], br, cre);
      cim = mm16(ar[s], bi, cim);
      cre = mm16(neg8(ai[s]), bi, cre);
      cim = mm16(ai[s], br, cim);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ky = drow(r, lh);
      if (ky < SKY && li < CH)
        gG[((long long)(ky * SKX + kx) * B + b) * SW + c0 + li] = f2{cre[r], cim[r]};
    }
  }
}

// The adjoint of the forward half:
//   out[b][i][y][x] = (Re sum_kx (sum_ky conj(fy[ky][y]) gH[b][m][i]) conj(fx[x][kx])
//                      + sum_o pw[i][o] gz[b][o][y][x]) GELU'(zp[b][i][y][x])
// (HEAD: the head's tables and 15 x 15 gF, no pointwise part; zp null: no
// GELU'). Block of 8 waves, grid (B, S): 4 / S of a patch's row groups y = 8 g ..
// + 7. Columns: per kx, D[y][i] over ky, straight from memory; rounded into LDS as
// rows [y][part][i] of 16 kx (zeros past the last), the operand of the rows:
// D[i][x] per y, a wave's row of each group.
template <bool HEAD, int S>
__global__ void __launch_bounds__(512) dft_fwd_adjoint_bf16(
    const f2* __restrict__ gH, const float* __restrict__ gz, const f2* __restrict__ fy,
    const f2* __restrict__ fx, const float* __restrict__ pw, const float* __restrict__ zp,
    float* __restrict__ out) {
  constexpr int KY = HEAD ? HN : SKY, KX = HEAD ? HN : SKX, KS = KY > 16 ? 2 : 1;
  constexpr int ROWS = SN / S;  // of this block
  __shared__ __attribute__((aligned(16))) __bf16 tt[ROWS][2][SW][16];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, li = lane & 31, lh = lane >> 5;
  const long long b = blockIdx.x;
  // the loads of the wave's first row (a row ahead below) and of the rows'
  // operands go out first: they are waited for after the columns
  float gv[16], zv[16];
  f2 xw[8];
  float pv[16];
  auto load_row = [&](int yl) {
    const int y = 8 * (yl / 8 * S + blockIdx.y) + wave;
    if constexpr (!HEAD)
#pragma unroll
      for (int j = 0; j < 16; ++j)
        gv[j] = gz[((b * SW + 16 * (j / 8) + 8 * lh + j % 8) * SN + y) * SN + li];
    if (zp)
#pragma unroll
      for (int r = 0; r < 16; ++r) zv[r] = zp[((b * SW + drow(r, lh)) * SN + y) * SN + li];
  };
  load_row(wave);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    xw[j] = fx[li * KX + min(8 * lh + j, KX - 1)];
    if constexpr (!HEAD) {
      pv[j] = pw[li * SW + 8 * lh + j];
      pv[8 + j] = pw[li * SW + 16 + 8 * lh + j];
    }
  }
  bf16x8 ar[KS], ai[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int ky = 16 * s + 8 * lh + j;
      const f2 w = fy[min(ky, KY - 1) * SN + li];
      ar[s][j] = (__bf16)(ky < KY ? w.x : 0.f);
      ai[s][j] = (__bf16)(ky < KY ? -w.y : 0.f);
    }
  // zeros past the last kx (kx = 8 of a layer is written over them below)
  for (int q = t; q < ROWS * 2 * SW; q += 512)
    *reinterpret_cast<u32x4*>(&(&tt[0][0][0][0])[q * 16 + 8]) = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  const f2* g0 = gH + b * KY * KX * SW + li;
  for (int kx = wave; kx < KX; kx += 8) {
    floatx16 cre = {0}, cim = {0};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      bf16x8 br, bi;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int ky = 16 * s + 8 * lh + j;
        f2 v = {0.f, 0.f};
        if (16 * s + j < KY) {  // (the second step holds ky = 16 alone)
          v = g0[(min(ky, KY - 1) * KX + kx) * SW];
          if (ky >= KY) v = f2{0.f, 0.f};
        }
        br[j] = (__bf16)v.x;
        bi[j] = (__bf16)v.y;
      }
      cre = mm16(ar[s], br, cre);
      cim = mm16(ar[s], bi, cim);
      cre = mm16(neg8(ai[s]), bi, cre);
      cim = mm16(ai[s], br, cim);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int g = r / 4;  // row group of y = drow(r, lh)
      if (S > 1 && g % S != (int)blockIdx.y) continue;
      const int yl = 8 * (g / S) + drow(r, lh) % 8;
      tt[yl][0][li][kx] = (__bf16)cre[r];
      tt[yl][1][li][kx] = (__bf16)cim[r];
    }
  }
  bf16x8 xr, xi, pa[2];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int kx = 8 * lh + j;
    xr[j] = (__bf16)(kx < KX ? xw[j].x : 0.f);
    xi[j] = (__bf16)(kx < KX ? -xw[j].y : 0.f);
    if constexpr (!HEAD) {
      pa[0][j] = (__bf16)pv[j];
      pa[1][j] = (__bf16)pv[8 + j];
    }
  }
  __syncthreads();
  for (int yl = wave; yl < ROWS; yl += 8) {
    const int y = 8 * (yl / 8 * S + blockIdx.y) + wave;
    const bf16x8 tr = *reinterpret_cast<const bf16x8*>(&tt[yl][0][li][8 * lh]);
    const bf16x8 ti = *reinterpret_cast<const bf16x8*>(&tt[yl][1][li][8 * lh]);
    floatx16 acc = {0}, accp = {0};
    if constexpr (!HEAD) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        bf16x8 g;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          g[j] = (__bf16)gv[8 * s + j];
        accp = mm16(pa[s], g, accp);
      }
    }
    acc = mm16(tr, xr, acc);
    acc = mm16(neg8(ti), xi, acc);
    float zc[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) zc[r] = zp ? zv[r] : 0.f;
    if (yl + 8 < ROWS) load_row(yl + 8);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const long long off = ((b * SW + drow(r, lh)) * SN + y) * SN + li;
      float v = acc[r];
      if constexpr (!HEAD) v += accp[r];
      if (zp) v *= gelu_grad_f(zc[r]);
      out[off] = v;
    }
  }
}

inline const f2* c2(const float* p) { return reinterpret_cast<const f2*>(p); }
inline f2* c2(float* p) { return reinterpret_cast<f2*>(p); }

}  // namespace

hipError_t sur_loss(const float* out, const float* tgt, long long n, float* part, float* sums,
                    float* g, hipStream_t s) {
  loss_chains<<<256 / LC, 256, 0, s>>>(out, tgt, n, part);
  loss_grad<<<(unsigned)((2 * n + 255) / 256), 256, 0, s>>>(out, tgt, part, sums, g, 2 * n);
  return hipGetLastError();
}

hipError_t sur_pointwise_grad(const float* h, const float* gz, int ci, int B, bool bf16,
                              float* part, float* out, SurSumJobs* sums, hipStream_t s) {
  const int units = 4 * B, nblk = std::min(units, kSurPointwiseParts), E = ci * SW + SW;
  auto go = [&](auto kern) { kern<<<nblk, 256, 0, s>>>(h, gz, units, part); };
  if (ci == 32) {
    if (bf16) go(pointwise_grad<true, 32>);
    else go(pointwise_grad<false, 32>);
  } else if (ci == 16) {
    if (bf16) go(pointwise_grad<true, 16>);
    else go(pointwise_grad<false, 16>);
  } else {
    return hipErrorInvalidValue;
  }
  sums->j[sums->n++] = {part, nblk, E, out};
  return hipGetLastError();
}

hipError_t sur_sum_parts(const SurSumJobs& jobs, hipStream_t s) {
  int blocks = 0;
  for (int q = 0; q < jobs.n; ++q) blocks += (jobs.j[q].E + 31) / 32;
  if (blocks) sum_parts<<<blocks, 256, 0, s>>>(jobs);
  return hipGetLastError();
}

hipError_t sur_spectral_grad(const float* H, const float* gG, int B, bool bf16, float* gW,
                             hipStream_t s) {
  if (bf16) spectral_grad<true><<<SNM, 256, 0, s>>>(c2(H), c2(gG), B, c2(gW));
  else spectral_grad<false><<<SNM, 256, 0, s>>>(c2(H), c2(gG), B, c2(gW));
  return hipGetLastError();
}

hipError_t sur_spec_from_mode_major(const float* gW, long long layer_stride_floats, int layers,
                                    float* G, hipStream_t s) {
  if (layer_stride_floats % 2 != 0) return hipErrorInvalidValue;
  spec_from_mode_major<<<dim3(SW, layers), 512, 0, s>>>(c2(gW), layer_stride_floats / 2, c2(G));
  return hipGetLastError();
}

hipError_t sur_head_grad(const float* F, const float* gout, int B, bool bf16, float* part,
                         float* out, SurSumJobs* sums, hipStream_t s) {
  const int slices = std::min(B, kSurHeadSlices), E = 2 * SW * OUT * HM;
  const dim3 grid((HM + 63) / 64, SW / 4, slices);
  if (bf16) head_grad<true><<<grid, 256, 0, s>>>(c2(F), c2(gout), B, c2(part));
  else head_grad<false><<<grid, 256, 0, s>>>(c2(F), c2(gout), B, c2(part));
  sums->j[sums->n++] = {part, slices, E, out};
  return hipGetLastError();
}

hipError_t sur_head_mix_adjoint_bf16(const float* gout, const float* head, int B, float* gF,
                                     hipStream_t s) {
  head_mix_adjoint_bf16<<<dim3((B + 31) / 32, (HM + 7) / 8), 512, 0, s>>>(c2(gout), c2(head), B,
                                                                          c2(gF));
  return hipGetLastError();
}
hipError_t sur_mode_mix_adjoint_bf16(const float* gG, const float* Wm, int B, float* gH,
                                     hipStream_t s) {
  mode_mix_adjoint_bf16<<<dim3((B + 31) / 32, (SNM + 3) / 4), 256, 0, s>>>(c2(gG), c2(Wm), B,
                                                                           c2(gH));
  return hipGetLastError();
}
// Splits of the two transforms' adjoints: as many as keep a launch within two
// blocks per CU. At 64 patches, 64 blocks took 29 us (forward half) and 11.9 us
// (inverse half), 256 blocks with their loads
// ahead of the tables 10.4 and 10.4.
hipError_t sur_dft_adjoint_bf16(const float* gz, const float* iy, const float* ix, int B,
                                float* gG, hipStream_t s) {
  auto go = [&](auto kern, int splits) {
    kern<<<dim3(B, splits), 512, 0, s>>>(gz, c2(iy), c2(ix), B, c2(gG));
  };
  if (B <= 128) go(dft_adjoint_bf16<4>, 4);
  else if (B <= 256) go(dft_adjoint_bf16<2>, 2);
  else go(dft_adjoint_bf16<1>, 1);
  return hipGetLastError();
}
hipError_t sur_dft_fwd_adjoint_bf16(const float* gH, const float* gz, const float* fy,
                                    const float* fx, const float* pw, const float* zp, bool head,
                                    int B, float* out, hipStream_t s) {
  auto go = [&](auto kern, int splits) {
    kern<<<dim3(B, splits), 512, 0, s>>>(c2(gH), gz, c2(fy), c2(fx), pw, zp, out);
  };
  if (head) {
    if (B <= 128) go(dft_fwd_adjoint_bf16<true, 4>, 4);
    else if (B <= 256) go(dft_fwd_adjoint_bf16<true, 2>, 2);
    else go(dft_fwd_adjoint_bf16<true, 1>, 1);
  } else {
    if (B <= 128) go(dft_fwd_adjoint_bf16<false, 4>, 4);
    else if (B <= 256) go(dft_fwd_adjoint_bf16<false, 2>, 2);
    else go(dft_fwd_adjoint_bf16<false, 1>, 1);
  }
  return hipGetLastError();
}

}  // namespace scw
