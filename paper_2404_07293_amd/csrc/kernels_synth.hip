// Field synthesis kernels, the hot path (Sec. 2.6, Sec. 4.1, Eqs. 9, 10, 30-34):
//
//   phase     W±[task][p][j] = a_j exp(i k g_j dz_top) ± b_j exp(-i k g_j dz_bot)
//   modal     spec[plane][r] = sum_j P_l[r][j] W(sign(r))[task][p][j]
//             (rows r < 2M are p_x, p_y and take W+, rows >= 2M are p_z and
//              take W-, because a forward/backward eigenvector pair shares
//              its E part and has opposite H parts)
//   exterior  spec of planes above / below the sample from the plane-wave
//             coefficients (Eq. 9)
//   idft      E[c][plane][g][f] = sum_{v,u} spec[plane][c][v][u]
//             exp(2 pi i (u f / fx + v g / fy)), as two passes (x, then y).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "scw_internal.h"

namespace scw {
namespace {

template <typename T>
struct cx {
  T x, y;
};

template <typename T>
__device__ __forceinline__ void cfma(cx<T>& acc, cx<T> a, cx<T> b) {
  acc.x = fma(a.x, b.x, acc.x);
  acc.x = fma(-a.y, b.y, acc.x);
  acc.y = fma(a.x, b.y, acc.y);
  acc.y = fma(a.y, b.x, acc.y);
}

struct zd {
  double x, y;
};
__device__ __forceinline__ zd zexp_i(zd arg) {  // exp(i * arg)
  double s, c;
  sincos(arg.x, &s, &c);
  double m = exp(-arg.y);
  return {m * c, m * s};
}
__device__ __forceinline__ zd zmul(zd a, zd b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

// ---------------------------------------------------------------- exterior
// Planes outside the sample. The modal sum's launch takes them as blocks after
// its own (they share no value with it; 150 x 90 x 45 points, a third of the
// planes outside: 14.0 us a call, 16.9 with a launch of their own);
// exterior_kernel is that launch where there is no modal sum or more than one
// volume.
struct ExtArgs {
  const ExtPlane* ext;
  const zd *coef, *ksz;
  int n_ext;
};
template <typename T>
__device__ inline void exterior_entry(const ExtArgs& x, long long t, int M,
                                      cx<T>* __restrict__ spec) {
  const int n3 = 3 * M;
  if (t >= (long long)x.n_ext * n3) return;
  const int r = (int)(t % n3);
  const ExtPlane e = x.ext[t / n3];
  const int m = r % M;
  zd val;
  if (e.kind == 0) {
    const zd kz = x.ksz[m];
    const zd gi = zexp_i({kz.x * e.dz, kz.y * e.dz});
    const zd gr = zexp_i({-kz.x * e.dz, -kz.y * e.dz});
    const zd pi = zmul(x.coef[r], gi), pr = zmul(x.coef[n3 + r], gr);
    val = {pi.x + pr.x, pi.y + pr.y};
  } else {
    const zd kz = x.ksz[M + m];
    val = zmul(x.coef[2 * n3 + r], zexp_i({kz.x * e.dz, kz.y * e.dz}));
  }
  spec[(long long)e.plane * n3 + r] = {(T)val.x, (T)val.y};
}

template <typename T>
__global__ void exterior_kernel(ExtArgs x, int M, long long spec_stride, cx<T>* __restrict__ spec) {
  x.coef += (long long)blockIdx.y * 9 * M;  // one volume (illumination) per blockIdx.y
  exterior_entry<T>(x, (long long)blockIdx.x * blockDim.x + threadIdx.x, M,
                    spec + blockIdx.y * spec_stride);
}

// ---------------------------------------------------------------- phase
// f = a g_f(z_p) and bk = b g_b(z_p) of plane p of a task.
__device__ __forceinline__ void phase_pair(zd g, zd a, zd b, const double* __restrict__ dzp, zd& f,
                                           zd& bk) {
  const zd gf = zexp_i({g.x * dzp[0], g.y * dzp[0]});
  const zd gb = zexp_i({-g.x * dzp[1], -g.y * dzp[1]});
  f = zmul(a, gf);
  bk = zmul(b, gb);
}

// One thread per (task, plane, column): the exponentials of a plane are a chain
// of some 300 dependent operations, so planes go side by side.
template <typename T>
__global__ void phase_kernel(const Task* __restrict__ tasks, const double* __restrict__ dz,
                             const zd* __restrict__ kg, const zd* __restrict__ a,
                             const zd* __restrict__ b, int n2, int zt, int ntasks,
                             cx<T>* __restrict__ w) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long long)ntasks * zt * n2) return;
  const int j = (int)(t % n2), p = (int)(t / n2 % zt), task = (int)(t / n2 / zt);
  const Task tk = tasks[task];
  cx<T> wp = {0, 0}, wm = {0, 0};
  if (p < tk.count) {
    const long long lj = (long long)tk.layer * n2 + j;
    zd f, bk;
    phase_pair(kg[lj], a[lj], b[lj], dz + ((long long)task * zt + p) * 2, f, bk);
    wp = {(T)(f.x + bk.x), (T)(f.y + bk.y)};
    wm = {(T)(f.x - bk.x), (T)(f.y - bk.y)};
  }
  w[(((long long)task * 2 + 0) * zt + p) * n2 + j] = wp;
  w[(((long long)task * 2 + 1) * zt + p) * n2 + j] = wm;
}

// ---------------------------------------------------------------- modal sum
// Sums over the lanes by recursive halving: v[i] of every lane summed in lane i
// (N - 1 shuffles for N values).
template <int N, typename T>
__device__ __forceinline__ void halve(T* v, int lane) {
  if constexpr (N > 1) {
    constexpr int H = N / 2;
    const bool up = (lane & H) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const T send = up ? v[i] : v[i + H];
      const T keep = up ? v[i + H] : v[i];
      v[i] = keep + __shfl_xor(send, H, 64);
    }
    halve<H>(v, lane);
  }
}

// One block = 4 waves; each wave owns RW consecutive rows of one category
// (x/y rows or z rows) of one task. The task's W table for that category is
// staged in LDS in chunks of jc columns (PH: computed there); lanes stride over
// j, every lane keeps RW x ZT partial sums, and halving over the lanes finishes
// them.
template <typename T, int ZT, int RW, bool PH>
__global__ void __launch_bounds__(256) modal_kernel(
    const cx<T>* __restrict__ P, const cx<T>* __restrict__ w, const zd* __restrict__ kg,
    const zd* __restrict__ a, const zd* __restrict__ b, const double* __restrict__ dz,
    const Task* __restrict__ tasks, int M, int nb_xy, int nb_z, int jc, int nmodal, ExtArgs x,
    cx<T>* __restrict__ spec) {
  constexpr int NV = 2 * RW * ZT;
  static_assert(NV <= 64 && (NV & (NV - 1)) == 0, "value count must be a power of two <= 64");
  if ((int)blockIdx.x >= nmodal) {
    exterior_entry<T>(x, (long long)(blockIdx.x - nmodal) * 256 + threadIdx.x, M, spec);
    return;
  }
  extern __shared__ unsigned char smem_raw[];
  cx<T>* sw = reinterpret_cast<cx<T>*>(smem_raw);  // [ZT][jc]
  const int n2 = 2 * M, n3 = 3 * M;
  const int nb = nb_xy + nb_z;
  const int task = blockIdx.x / nb;
  const int rb = blockIdx.x % nb;
  const Task tk = tasks[task];
  const int sign = rb < nb_xy ? 0 : 1;
  const int rows_per_block = 4 * RW;
  const int row_begin = sign == 0 ? rb * rows_per_block : n2 + (rb - nb_xy) * rows_per_block;
  const int row_end = sign == 0 ? n2 : n3;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r0 = row_begin + wave * RW;
  const cx<T>* Pl = P + (long long)tk.layer * n3 * n2;
  const cx<T>* wt = PH ? nullptr : w + ((long long)task * 2 + sign) * ZT * n2;

  T acc[NV];  // [r][p][re, im]
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0;

  // rows one step ahead, the first step's while the table is filled (indices
  // past the last row or column are clamped; their sums are not used)
  const cx<T>* prow[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) prow[r] = Pl + (long long)min(r0 + r, row_end - 1) * n2;
  cx<T> nxt[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) nxt[r] = prow[r][min(lane, n2 - 1)];

  for (int j0 = 0; j0 < n2; j0 += jc) {
    const int jn = min(jc, n2 - j0);
    if (j0 > 0) __syncthreads();
    for (int i = threadIdx.x; i < ZT * jn; i += blockDim.x) {
      const int p = i / jn, jj = i % jn;
      if constexpr (PH) {
        cx<T> v = {0, 0};
        if (p < tk.count) {
          const long long lj = (long long)tk.layer * n2 + j0 + jj;
          zd f, bk;
          phase_pair(kg[lj], a[lj], b[lj], dz + ((long long)task * ZT + p) * 2, f, bk);
          v = sign == 0 ? cx<T>{(T)(f.x + bk.x), (T)(f.y + bk.y)}
                        : cx<T>{(T)(f.x - bk.x), (T)(f.y - bk.y)};
        }
        sw[p * jc + jj] = v;
      } else {
        sw[p * jc + jj] = wt[(long long)p * n2 + j0 + jj];
      }
    }
    __syncthreads();
    for (int jj = lane; jj < jn; jj += 64) {
      // the next step of this chunk, or the first of the next one
      const int jq = jj + 64 < jn ? j0 + jj + 64 : j0 + jn + lane;
      cx<T> wv[ZT], cur[RW];
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        cur[r] = nxt[r];
        nxt[r] = prow[r][min(jq, n2 - 1)];
      }
#pragma unroll
      for (int p = 0; p < ZT; ++p) wv[p] = sw[p * jc + jj];
#pragma unroll
      for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int p = 0; p < ZT; ++p) {
          cx<T> s = {acc[(r * ZT + p) * 2], acc[(r * ZT + p) * 2 + 1]};
          cfma(s, cur[r], wv[p]);
          acc[(r * ZT + p) * 2] = s.x;
          acc[(r * ZT + p) * 2 + 1] = s.y;
        }
    }
  }
  halve<NV>(acc, lane);
#pragma unroll
  for (int off = NV; off < 64; off <<= 1) acc[0] += __shfl_xor(acc[0], off, 64);
  if (lane < NV) {
    const int p = (lane >> 1) % ZT, row = r0 + (lane >> 1) / ZT;
    if (row < row_end && p < tk.count)
      reinterpret_cast<T*>(spec)[((long long)(tk.plane0 + p) * n3 + row) * 2 + (lane & 1)] = acc[0];
  }
}

// ---------------------------------------------------------------- modal sum, FP32
// Phase factors are generated in the block: W(sign)[p][j] = a_j g_f(z_p) +-
// b_j g_b(z_p) for the block's rows' sign, written straight into LDS. Lanes
// read P two complex at a time (16-byte loads); every lane accumulates
// RW rows x ZT planes, and a recursive-halving butterfly leaves the complete
// sum of value index i in lane i (NV = 2 RW ZT values, NV - 1 shuffles).
// Bound by the read of P where there are many layers: 300 MB (32 layers, M = 441)
// take 52.6 us (5.7 TB/s; a plain read of them 43.4), 56 with the loads one step
// ahead and begun after the phases; by its prologue (phases, first loads) where
// there are few: 39 MB (16 layers, M = 225) take 10.3 us, 12.5 before.
// exp(i (re + i im)) for the phase factors of the FP32 modal sum. The angle is
// first reduced to [-pi, pi] by Cody and Waite's two-constant subtraction of
// the nearest multiple of 2 pi, then passed to the hardware sine and cosine;
// the magnitude uses the hardware exponential. The absolute phase error stays
// near 1e-6 for the angles k gamma dz of a layer (up to a few hundred
// radians), well inside the FP32 path's budget, at a fraction of the cost of
// the correctly rounded functions (these factors are rebuilt by every block).
__device__ __forceinline__ float2 cexpi_f(float re, float im) {
  const float n = rintf(re * 0.159154943091895336f);  // re / (2 pi), nearest integer
  float r = fmaf(-n, 6.28318548202514648f, re);       // 2 pi rounded to float
  r = fmaf(n, 1.74845553e-7f, r);                     // minus its rounding error
  const float m = __expf(-im);
  return make_float2(m * __cosf(r), m * __sinf(r));
}

template <int ZT, int RW>
__global__ void __launch_bounds__(256) modal_f32_kernel(
    const float4* __restrict__ P, const float2* __restrict__ kgab, const Task* __restrict__ tasks,
    const float2* __restrict__ tdz, int M, int L, int nb_xy, int nb_z, int jc, int nmodal,
    ExtArgs x, float2* __restrict__ spec) {
  constexpr int NV = 2 * RW * ZT;
  static_assert(NV <= 64 && (NV & (NV - 1)) == 0, "value count must be a power of two <= 64");
  if ((int)blockIdx.x >= nmodal) {
    exterior_entry<float>(x, (long long)(blockIdx.x - nmodal) * 256 + threadIdx.x, M,
                          reinterpret_cast<cx<float>*>(spec));
    return;
  }
  extern __shared__ float4 sw4[];  // [ZT][jc / 2]
  float2* sw = reinterpret_cast<float2*>(sw4);
  const int n2 = 2 * M, n3 = 3 * M, h2 = M;  // h2 = float4 per row
  const int nb = nb_xy + nb_z;
  const int task = blockIdx.x / nb;
  const int rb = blockIdx.x % nb;
  const Task tk = tasks[task];
  const bool zrows = rb >= nb_xy;
  const int rows_per_block = 4 * RW;
  const int row_begin = zrows ? n2 + (rb - nb_xy) * rows_per_block : rb * rows_per_block;
  const int row_end = zrows ? n3 : n2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r0 = row_begin + wave * RW;
  const float4* Pl = P + (long long)tk.layer * n3 * h2;
  const float2* kg = kgab + (long long)tk.layer * n2;
  const float2* av = kgab + ((long long)L + tk.layer) * n2;
  const float2* bv = kgab + (2LL * L + tk.layer) * n2;
  const float sgn = zrows ? -1.f : 1.f;
  const char* prow[RW];  // wave-uniform: loads take a scalar base and a 32-bit offset
#pragma unroll
  for (int r = 0; r < RW; ++r)
    prow[r] = reinterpret_cast<const char*>(Pl + (long long)min(r0 + r, row_end - 1) * h2);
  float2 dzp[ZT];
#pragma unroll
  for (int p = 0; p < ZT; ++p) dzp[p] = tdz[task * ZT + p];

  // The phase table holds jq float4 per plane, jq = jc / 2 rounded up to a
  // multiple of 64, with zeros past the chunk. Every lane then runs the same
  // ceil(qn / 64) steps: a lane past the chunk reads a valid element of its
  // row (the index clamped to the row) and adds its product with a zero
  // weight, which leaves its sums unchanged. The loads run two steps ahead, in
  // two register sets: both are filled before the phases are computed, and a
  // step loads its successor's successor into each row's registers as soon as
  // that row's products are done. Loads return in order, so those of the first
  // phases go out before the rows', and the rows' in the order of their use
  // (the barriers of the scheduler keep both).
  const int jq = (jc / 2 + 63) / 64 * 64;
  constexpr int KG = 4;  // phase arguments loaded ahead: the first 1024
  float2 kgr[KG], avr[KG], bvr[KG];
#pragma unroll
  for (int k = 0; k < KG; ++k) {
    const int j = min((int)threadIdx.x + 256 * k, n2 - 1);
    kgr[k] = kg[j];
    avr[k] = av[j];
    bvr[k] = bv[j];
  }
  auto phases = [&](int jj, int jn, float2 g, float2 a, float2 b) {
    if (jj < jn) {
#pragma unroll
      for (int p = 0; p < ZT; ++p) {
        const float2 gf = cexpi_f(g.x * dzp[p].x, g.y * dzp[p].x);
        const float2 gb = cexpi_f(-g.x * dzp[p].y, -g.y * dzp[p].y);
        const float fx = a.x * gf.x - a.y * gf.y, fy = a.x * gf.y + a.y * gf.x;
        const float bx = b.x * gb.x - b.y * gb.y, by = b.x * gb.y + b.y * gb.x;
        sw[p * 2 * jq + jj] = make_float2(fx + sgn * bx, fy + sgn * by);
      }
    } else if (jj < 2 * jq) {
#pragma unroll
      for (int p = 0; p < ZT; ++p) sw[p * 2 * jq + jj] = make_float2(0.f, 0.f);
    }
  };
  auto load = [&](int r, int q) {
    return *reinterpret_cast<const float4*>(prow[r] + 16u * (unsigned)min(q, h2 - 1));
  };
  __builtin_amdgcn_sched_barrier(0);
  float4 pa[RW], pb[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    pa[r] = load(r, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    pb[r] = load(r, lane + 64);
    __builtin_amdgcn_sched_barrier(0);
  }
  auto more_phases = [&](int j0, int jn, int from) {
    for (int jj = threadIdx.x + from; jj < 2 * jq; jj += 256) {
      const int j = min(j0 + jj, n2 - 1);
      phases(jj, jn, kg[j], av[j], bv[j]);
    }
  };
#pragma unroll
  for (int k = 0; k < KG; ++k)  // a use here: the loads above stay above
    asm volatile("" : "+v"(kgr[k].x), "+v"(kgr[k].y), "+v"(avr[k].x), "+v"(avr[k].y),
                      "+v"(bvr[k].x), "+v"(bvr[k].y));
#pragma unroll
  for (int k = 0; k < KG; ++k)
    phases(threadIdx.x + 256 * k, min(jc, n2), kgr[k], avr[k], bvr[k]);
  more_phases(0, min(jc, n2), 256 * KG);
  float acc[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) acc[i] = 0.f;
  auto step = [&](float4 (&cur)[RW], int q, int qg) {
    float4 w[ZT];
#pragma unroll
    for (int p = 0; p < ZT; ++p) w[p] = sw4[p * jq + q];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
#pragma unroll
      for (int p = 0; p < ZT; ++p) {
        float& re = acc[(r * ZT + p) * 2];
        float& im = acc[(r * ZT + p) * 2 + 1];
        re = fmaf(cur[r].x, w[p].x, re);
        re = fmaf(-cur[r].y, w[p].y, re);
        im = fmaf(cur[r].x, w[p].y, im);
        im = fmaf(cur[r].y, w[p].x, im);
        re = fmaf(cur[r].z, w[p].z, re);
        re = fmaf(-cur[r].w, w[p].w, re);
        im = fmaf(cur[r].z, w[p].w, im);
        im = fmaf(cur[r].w, w[p].z, im);
      }
      cur[r] = load(r, qg);
      // keep the load here (the scheduler would otherwise sink it)
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int j0 = 0; j0 < n2; j0 += jc) {
    const int jn = min(jc, n2 - j0);
    if (j0 > 0) {
      __syncthreads();
      more_phases(j0, jn, 0);
    }
    __syncthreads();
    // step i covers q = lane + 64 i of the chunk and loads element q + 128 of
    // the rows, which may belong to the next chunk: a chunk before the last has
    // jc / 128 steps, an even number, so the sets keep their turns
    const int q0 = j0 / 2, ns = (jn / 2 + 63) / 64;
    int i = 0;
    for (; i + 2 <= ns; i += 2) {
      const int q = lane + 64 * i;
      step(pa, q, q0 + q + 128);
      step(pb, q + 64, q0 + q + 192);
    }
    if (i < ns) step(pa, lane + 64 * i, h2 - 1);
  }
  halve<NV>(acc, lane);
#pragma unroll
  for (int off = NV; off < 64; off <<= 1) acc[0] += __shfl_xor(acc[0], off, 64);
  if (lane < NV) {
    const int comp = lane & 1, p = (lane >> 1) % ZT, r = (lane >> 1) / ZT;
    const int row = r0 + r;
    if (row < row_end && p < tk.count)
      reinterpret_cast<float*>(spec)[((long long)(tk.plane0 + p) * n3 + row) * 2 + comp] = acc[0];
  }
}

template <int ZT, int RW>
hipError_t launch_modal_f32_rw(const SynthArgs& a, hipStream_t s, const ExtArgs& x) {
  const int n2 = 2 * a.M;
  const int rows_per_block = 4 * RW;
  const int nb_xy = (n2 + rows_per_block - 1) / rows_per_block;
  const int nb_z = (a.M + rows_per_block - 1) / rows_per_block;
  const size_t max_lds = 64 * 1024;
  int jc = (int)(max_lds / (ZT * sizeof(float2)));
  jc = jc >= n2 ? n2 : (jc / 128) * 128;
  // per plane jc / 2 float4 of phases, padded with zeros to a multiple of 64
  const size_t lds = (size_t)ZT * ((jc / 2 + 63) / 64 * 64) * sizeof(float4);
  const long long nblocks = (long long)a.ntasks * (nb_xy + nb_z);
  if (nblocks == 0) return hipSuccess;
  const long long ext = ((long long)x.n_ext * 3 * a.M + 255) / 256;
  modal_f32_kernel<ZT, RW><<<(unsigned)(nblocks + ext), 256, lds, s>>>(
      reinterpret_cast<const float4*>(a.P), reinterpret_cast<const float2*>(a.kgab32), a.tasks,
      reinterpret_cast<const float2*>(a.task_dz32), a.M, a.L, nb_xy, nb_z, jc, (int)nblocks, x,
      reinterpret_cast<float2*>(a.spec));
  return hipGetLastError();
}

// Rows per wave RW with 2 RW ZT <= 64 accumulated values per lane.
template <int ZT>
hipError_t launch_modal_f32(const SynthArgs& a, hipStream_t s, const ExtArgs& x) {
  switch (a.modal_rw) {
    case 2: return launch_modal_f32_rw<ZT, 2>(a, s, x);
    case 4: return launch_modal_f32_rw<ZT, 4>(a, s, x);
    case 8:
      if constexpr (ZT <= 4) return launch_modal_f32_rw<ZT, 8>(a, s, x);
      break;
    case 16:
      if constexpr (ZT <= 2) return launch_modal_f32_rw<ZT, 16>(a, s, x);
      break;
    default: break;
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- modal sum, many illuminations
// With several illuminations the columns of a task are (illumination, plane)
// pairs c = ki * zt + p, 32 per launch group, and the product P_l W becomes a
// real GEMM pair on the matrix cores: spec_re = P_re W_re - P_im W_im and
// spec_im = P_re W_im + P_im W_re, in v_mfma_f32_16x16x4f32 (lane l holds row
// or column l % 16 of K slot l / 16; accumulator i is D[4 (l / 16) + i][l % 16]).
//
// K goes in steps of 16 j: in its s-th product (s < 4) slot g stands for j =
// step + 4 g + s, so that a lane reads four consecutive complex of its row of P
// (32 bytes; the four slots a 128-byte run) and four of its column of W.
// multi_phase_kernel writes the group's phase table once, W = a_kj g_f(z_p) +-
// b_kj g_b(z_p), zero for j >= 2M and for columns past the group, in the order in
// which the products read it: [task][sign][step][half of the columns][half of a
// lane's four][lane] pairs of complex, so that a wave's load is 1 KB in a row.
//
// modal_multi_kernel: one block = four waves on the same 16 rows of one sign
// category of one task. Wave w takes steps w, w + 4, ...; its operands come
// straight from memory, two steps ahead, and no wave waits for another before the
// four tiles are added through LDS. Bound by the FP32 matrix rate once the chip
// is filled evenly (16 tasks at M = 225: 9 us of products, in 736 blocks of 16
// rows): 19.3 us with its 39 MB of P, 23.9 in blocks of 32 rows with the operands
// staged through LDS, 24.9 with eight waves per block.
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ void multi_phase_kernel(const float2* __restrict__ kg, const float2* __restrict__ ab,
                                   const Task* __restrict__ tasks,
                                   const float2* __restrict__ tdz, int zt, int M, int L, int n2p,
                                   int k0, int kcount, int ntasks, float2* __restrict__ W) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int per_task = 32 * n2p;
  if (t >= (long long)ntasks * per_task) return;
  const int task = (int)(t / per_task);
  const int rem = (int)(t % per_task);  // (step, column half, s / 2, lane, s % 2)
  const int lane = (rem >> 1) & 63;
  const int c = ((rem >> 8) & 1) * 16 + (lane & 15);
  const int j = (rem >> 9) * 16 + 4 * (lane >> 4) + ((rem >> 7) & 1) * 2 + (rem & 1);
  const int ki = c / zt, p = c % zt;
  const int n2 = 2 * M;
  float2 wp = make_float2(0.f, 0.f), wm = wp;
  if (j < n2 && ki < kcount) {
    const int layer = tasks[task].layer;
    const float2 g = kg[(long long)layer * n2 + j];
    const float2 dz = tdz[task * zt + p];
    const float2 gf = cexpi_f(g.x * dz.x, g.y * dz.x);
    const float2 gb = cexpi_f(-g.x * dz.y, -g.y * dz.y);
    const float2* abk = ab + (long long)(k0 + ki) * 2 * L * n2;
    const float2 a = abk[(long long)layer * n2 + j];
    const float2 b = abk[((long long)L + layer) * n2 + j];
    const float fx = a.x * gf.x - a.y * gf.y, fy = a.x * gf.y + a.y * gf.x;
    const float bx = b.x * gb.x - b.y * gb.y, by = b.x * gb.y + b.y * gb.x;
    wp = make_float2(fx + bx, fy + by);
    wm = make_float2(fx - bx, fy - by);
  }
  W[((long long)task * 2 + 0) * per_task + rem] = wp;
  W[((long long)task * 2 + 1) * per_task + rem] = wm;
}

__global__ void __launch_bounds__(256) modal_multi_kernel(
    const float4* __restrict__ P, const float4* __restrict__ W, const Task* __restrict__ tasks,
    int zt, int M, int fz, int n2p, int k0, int kcount, int ntasks, int nb_xy, int nb_z,
    float2* __restrict__ spec) {
  __shared__ float red[4][16][64];  // the waves' tiles: [wave][i, column half, part][lane]
  const int n2 = 2 * M, n3 = 3 * M;
  const int nb = nb_xy + nb_z;
  // Consecutive workgroups go to the eight XCDs in turn; numbering them so
  // that XCD x runs the logical blocks [x per, (x + 1) per) keeps a task's
  // blocks, which all read that task's W, on one XCD and its L2. The grid is
  // padded to 8 per blocks; the padding exits at once.
  const int per = gridDim.x / 8;
  const int blk = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (blk >= ntasks * nb) return;
  const int task = blk / nb;
  const int rb = blk % nb;
  const Task tk = tasks[task];
  const bool zrows = rb >= nb_xy;
  const int r0 = zrows ? n2 + (rb - nb_xy) * 16 : rb * 16;
  const int row_end = zrows ? n3 : n2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lg = lane >> 4;
  // rows past the end repeat the last one; j past 2M meets zero entries of W, so
  // P there only has to be finite and its index is clamped to the row's last pair
  const float4* prow = P + ((long long)tk.layer * n3 + min(r0 + li, row_end - 1)) * (n2 / 2);
  const float4* wt = W + ((long long)task * 2 + (zrows ? 1 : 0)) * 16 * n2p;
  const int pmax = n2 / 2 - 1, nsteps = n2p / 16;
  struct Set {
    float4 p[2], w[2][2];  // [half of the four], [column half][half of the four]
  };
  auto load = [&](Set& o, int i) {  // step wave + 4 i (the last step's again past the end)
    const int st = min(wave + 4 * i, nsteps - 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      o.p[h] = prow[min(8 * st + 2 * lg + h, pmax)];
#pragma unroll
      for (int c = 0; c < 2; ++c) o.w[c][h] = wt[st * 256 + (2 * c + h) * 64 + lane];
    }
  };
  // three accumulators per column half, so that no operand needs a sign flip:
  // spec_re = rr - ii, spec_im = im
  f32x4 rr[2], ii[2], im[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) rr[c] = ii[c] = im[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](Set& o, int i) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 a = o.p[h];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const float4 b = o.w[c][h];
        rr[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, rr[c], 0, 0, 0);
        ii[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, ii[c], 0, 0, 0);
        im[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.y, im[c], 0, 0, 0);
        rr[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, rr[c], 0, 0, 0);
        ii[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, ii[c], 0, 0, 0);
        im[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.x, im[c], 0, 0, 0);
        im[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.w, im[c], 0, 0, 0);
        im[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.z, im[c], 0, 0, 0);
      }
    }
    load(o, i + 2);
    __builtin_amdgcn_sched_barrier(0);
  };
  Set s0, s1;
  load(s0, 0);
  __builtin_amdgcn_sched_barrier(0);
  load(s1, 1);
  __builtin_amdgcn_sched_barrier(0);
  const int mine = (nsteps - wave + 3) / 4;
  int i = 0;
  for (; i + 2 <= mine; i += 2) {
    step(s0, i);
    step(s1, i + 1);
  }
  if (i < mine) step(s0, i);
  // the four waves' tiles are added through LDS, wave w the rows 4 g + w
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[wave][4 * r + 2 * c][lane] = rr[c][r] - ii[c][r];
      red[wave][4 * r + 2 * c + 1][lane] = im[c][r];
    }
  __syncthreads();
  const int row = r0 + 4 * lg + wave;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    float x = 0.f, y = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      x += red[w][4 * wave + 2 * c][lane];
      y += red[w][4 * wave + 2 * c + 1][lane];
    }
    const int col = 16 * c + li, ki = col / zt, p = col % zt;
    if (row < row_end && ki < kcount && p < tk.count)
      spec[((long long)(k0 + ki) * fz + tk.plane0 + p) * n3 + row] = make_float2(x, y);
  }
}

// ---------------------------------------------------------------- inverse DFT
// One block per (plane, component, f tile, g tile). The spectrum S[v][u] of the
// plane/component is staged in LDS; each thread owns one output column f:
//   pass x:  T[v][f] = sum_u S[v][u] exp(2 pi i u f / fx)
//            = e^{-2 pi i (U/2) f/fx} * Horner_u(S[v][.], w_f),  w_f = e^{2 pi i f/fx}
//            kept in LDS as T[v][thread];
//   pass y:  E[g][f] = e^{-2 pi i (V/2) g/fy} * Horner_v(T[.][f], w_g)
//            for the block's rows g, four rows at a time sharing each LDS read.
// wx[0][f] = w_f, wx[1][f] = e^{-2 pi i (U/2) f/fx}; wy likewise for g.
template <typename T>
__device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ __forceinline__ cx<T> cmuladd(cx<T> a, cx<T> w, cx<T> c) {  // a*w + c
  cx<T> r;
  r.x = fma(a.x, w.x, fma(-a.y, w.y, c.x));
  r.y = fma(a.x, w.y, fma(a.y, w.x, c.y));
  return r;
}

template <typename T, int FT>
__global__ void __launch_bounds__(FT) idft_kernel(
    const cx<T>* __restrict__ spec, const cx<T>* __restrict__ wx, const cx<T>* __restrict__ wy,
    int U, int V, int fx, int fy, int fz, int grows, cx<T>* __restrict__ E) {
  extern __shared__ unsigned char smem_raw[];
  cx<T>* S = reinterpret_cast<cx<T>*>(smem_raw);  // [V*U]
  cx<T>* Tt = S + U * V;                          // [V][FT]
  const int M = U * V;
  const int pc = blockIdx.z;
  const int plane = pc / 3, comp = pc % 3;
  const int t = threadIdx.x;
  const int f = blockIdx.x * FT + t;
  const int g0 = blockIdx.y * grows;
  const int g1 = min(fy, g0 + grows);
  const cx<T>* src = spec + ((long long)plane * 3 + comp) * M;
  for (int i = t; i < M; i += FT) S[i] = src[i];
  __syncthreads();
  const bool live = f < fx;
  if (live) {
    const cx<T> w = wx[f], sh = wx[fx + f];
    for (int v = 0; v < V; ++v) {
      const cx<T>* row = S + v * U;
      cx<T> acc = row[U - 1];
      for (int u = U - 2; u >= 0; --u) acc = cmuladd(acc, w, row[u]);
      Tt[v * FT + t] = cmul(acc, sh);
    }
  }
  // each thread reads only its own column of Tt: no barrier needed
  if (!live) return;
  cx<T>* dst = E + (((long long)comp * fz + plane) * fy) * fx + f;
  int g = g0;
  for (; g + 4 <= g1; g += 4) {
    cx<T> w[4], acc[4];
    const cx<T> top = Tt[(V - 1) * FT + t];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      w[k] = wy[g + k];
      acc[k] = top;
    }
    for (int v = V - 2; v >= 0; --v) {
      const cx<T> c = Tt[v * FT + t];
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] = cmuladd(acc[k], w[k], c);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const cx<T> o = cmul(acc[k], wy[fy + g + k]);
      __builtin_nontemporal_store(o.x, &dst[(long long)(g + k) * fx].x);
      __builtin_nontemporal_store(o.y, &dst[(long long)(g + k) * fx].y);
    }
  }
  for (; g < g1; ++g) {
    const cx<T> w = wy[g];
    cx<T> acc = Tt[(V - 1) * FT + t];
    for (int v = V - 2; v >= 0; --v) acc = cmuladd(acc, w, Tt[v * FT + t]);
    const cx<T> o = cmul(acc, wy[fy + g]);
    __builtin_nontemporal_store(o.x, &dst[(long long)g * fx].x);
    __builtin_nontemporal_store(o.y, &dst[(long long)g * fx].y);
  }
}

// ---------------------------------------------------------------- inverse DFT, factored
// For fy = R * P with P in {2, 4, 8, 16, 32} and V <= 32. One block per
// (plane/component, 64 columns f); threads are 64 columns x 4 groups.
//   x pass: T[v][f] by Horner (as above) into 32 zero-padded slots s = v + 16.
//   y pass: write g = g1 + R g2. With w = exp(2 pi i / fy), w^R = exp(2 pi i / P):
//     E[g1 + R g2] = sum_r A[r] exp(2 pi i r g2 / P),
//     A[r] = sum_{v = r mod P} T[v] w^(v g1),
//   so each (column, g1) costs 32 twiddle MACs plus one P-point FFT held in
//   registers, and writes P outputs; each store writes 64 consecutive columns.
// cos(2 pi r / 32) for r = 0..8: the first quadrant of the twiddles of every
// radix P <= 32 (e^{2 pi i k / P} is entry k * 32 / P of the full circle).
__device__ __forceinline__ double quarter_cos(int r) {
  switch (r) {
    case 0: return 1.0;
    case 1: return 0.98078528040323044913;
    case 2: return 0.92387953251128675613;
    case 3: return 0.83146961230254523708;
    case 4: return 0.70710678118654752440;
    case 5: return 0.55557023301960222474;
    case 6: return 0.38268343236508977173;
    case 7: return 0.19509032201612826785;
    default: return 0.0;
  }
}

// v * e^{2 pi i k / P} for a k known at compile time once the caller's loops
// are unrolled: no multiply for k = 0, a swap for the quarter turn, and the
// constant folded in otherwise.
template <typename T, int P>
__device__ __forceinline__ cx<T> twiddle_mul(cx<T> v, int k) {
  const int k32 = (k * (32 / P)) & 31;
  if (k32 == 0) return v;
  if (k32 == 8) return {-v.y, v.x};
  if (k32 == 16) return {-v.x, -v.y};
  if (k32 == 24) return {v.y, -v.x};
  const int q = k32 >> 3, r = k32 & 7;
  const T c0 = (T)quarter_cos(r), s0 = (T)quarter_cos(8 - r);
  const T c = q == 0 ? c0 : (q == 1 ? -s0 : (q == 2 ? -c0 : s0));
  const T sn = q == 0 ? s0 : (q == 1 ? c0 : (q == 2 ? -s0 : -c0));
  return {v.x * c - v.y * sn, v.x * sn + v.y * c};
}

// In-register radix-2 FFT of length P with positive exponent:
// a[g2] <- sum_r a[r] e^{2 pi i r g2 / P}.
template <typename T, int P>
__device__ __forceinline__ void small_fft(cx<T>* a) {
  // bit-reversal permutation
#pragma unroll
  for (int i = 0; i < P; ++i) {
    int r = 0;
#pragma unroll
    for (int b = 1, x = i; b < P; b <<= 1, x >>= 1) r = (r << 1) | (x & 1);
    if (r > i) {
      const cx<T> tmp = a[i];
      a[i] = a[r];
      a[r] = tmp;
    }
  }
#pragma unroll
  for (int len = 2; len <= P; len <<= 1) {
#pragma unroll
    for (int i = 0; i < P; i += len) {
#pragma unroll
      for (int j = 0; j < len / 2; ++j) {
        const cx<T> u = a[i + j];
        const cx<T> t = twiddle_mul<T, P>(a[i + j + len / 2], j * (P / len));
        a[i + j] = {u.x + t.x, u.y + t.y};
        a[i + j + len / 2] = {u.x - t.x, u.y - t.y};
      }
    }
  }
}

// One non-temporal store of a whole complex value (the field is written once
// and not read back by the synthesis).
__device__ __forceinline__ void store_nt(cx<float>* d, cx<float> v) {
  typedef float f2v __attribute__((ext_vector_type(2)));
  __builtin_nontemporal_store(f2v{v.x, v.y}, reinterpret_cast<f2v*>(d));
}
__device__ __forceinline__ void store_nt(cx<double>* d, cx<double> v) {
  typedef double d2v __attribute__((ext_vector_type(2)));
  __builtin_nontemporal_store(d2v{v.x, v.y}, reinterpret_cast<d2v*>(d));
}

// COLS columns per block (64 or 32); the 256 threads are COLS columns x
// 256 / COLS groups, each group taking every (256 / COLS)-th row in the x
// pass and g1 value in the y pass. The occupied frequency slots are lo..hi
// (slot = v + 16); the y pass runs over rounds of P slots that start at
// multiples of P, so that a slot's residue (slot - 16) mod P is fixed at
// compile time, and the slots of those rounds outside lo..hi hold zeros.
template <typename T, int P, int COLS>
__global__ void __launch_bounds__(256) idft_fft_kernel(
    const cx<T>* __restrict__ spec, const cx<T>* __restrict__ wx, const cx<T>* __restrict__ tw1g,
    int U, int V, int fx, int fy, int fz, cx<T>* __restrict__ E) {
  constexpr int NG = 256 / COLS;
  extern __shared__ unsigned char smem_raw[];
  const int R = fy / P;
  cx<T>* S = reinterpret_cast<cx<T>*>(smem_raw);  // [V*U]
  cx<T>* Ts = S + U * V;                          // [32][COLS]
  cx<T>* tw1 = Ts + 32 * COLS;                    // [R][32]: w^((s-16) g1)
  const int M = U * V;
  const int pc = blockIdx.y;
  const int plane = pc / 3, comp = pc % 3;
  const int t = threadIdx.x, col = t % COLS, q = t / COLS;
  const int f = blockIdx.x * COLS + col;
  const bool live = f < fx;
  const int lo = 16 - V / 2, hi = 16 + V / 2;
  const int s_begin = (lo / P) * P, s_end = (hi / P + 1) * P;
  const cx<T>* src = spec + (long long)pc * M;
  for (int i = t; i < M; i += 256) S[i] = src[i];
  for (int i = t; i < 32 * R; i += 256) tw1[i] = tw1g[i];
  {
    const int zl = lo - s_begin, zh = s_end - hi - 1;
    for (int i = t; i < (zl + zh) * COLS; i += 256) {
      const int rr = i / COLS, cc = i % COLS;
      const int sl = rr < zl ? s_begin + rr : hi + 1 + (rr - zl);
      Ts[sl * COLS + cc] = {0, 0};
    }
  }
  __syncthreads();
  if (live) {
    const cx<T> w = wx[f], sh = wx[fx + f];
    for (int vi = q; vi < V; vi += NG) {
      const cx<T>* row = S + vi * U;
      cx<T> acc = row[U - 1];
      for (int u = U - 2; u >= 0; --u) acc = cmuladd(acc, w, row[u]);
      Ts[(vi - V / 2 + 16) * COLS + col] = cmul(acc, sh);
    }
  }
  __syncthreads();
  if (!live) return;
  const cx<T>* tc = Ts + col;
  cx<T>* dst = E + (((long long)comp * fz + plane) * fy) * fx + f;
  const long long step = (long long)R * fx;
  for (int g1 = q; g1 < R; g1 += NG) {
    const cx<T>* tw = tw1 + g1 * 32;
    cx<T> a[P];
#pragma unroll
    for (int r = 0; r < P; ++r) a[r] = {0, 0};
    for (int s0 = s_begin; s0 < s_end; s0 += P) {
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const int r = (i - 16) & (P - 1);
        const cx<T> tv = tc[(s0 + i) * COLS], w1 = tw[s0 + i];
        a[r].x = fma(tv.x, w1.x, fma(-tv.y, w1.y, a[r].x));
        a[r].y = fma(tv.x, w1.y, fma(tv.y, w1.x, a[r].y));
      }
    }
    small_fft<T, P>(a);
    cx<T>* d = dst + (long long)g1 * fx;  // row g1 + R g2
#pragma unroll
    for (int g2 = 0; g2 < P; ++g2) store_nt(d + g2 * step, a[g2]);
  }
}

// ---------------------------------------------------------------- lateral slice
// Eq. 10 on an x-z (axis 0) or y-z (axis 1) plane. One block per plane and
// component: the spectrum's other lateral index is summed first with the
// phase of the slice position, T[k] = sum_j S e^{2 pi i (j - J/2) frac}
// (in FP64; the J phases per block are few), then the kept index runs on the
// n samples by Horner's rule as in the volume's x pass.
template <typename T>
__global__ void __launch_bounds__(256) slice_kernel(const cx<T>* __restrict__ spec,
                                                    const cx<T>* __restrict__ tw, int U, int V,
                                                    int n, int fz, int axis, double frac,
                                                    cx<T>* __restrict__ E) {
  extern __shared__ unsigned char smem_raw[];
  cx<T>* S = reinterpret_cast<cx<T>*>(smem_raw);  // [V][U]
  cx<T>* Tk = S + U * V;                          // [K]
  const int M = U * V, pc = blockIdx.x;
  const cx<T>* src = spec + (long long)pc * M;
  for (int i = threadIdx.x; i < M; i += blockDim.x) S[i] = src[i];
  __syncthreads();
  const int K = axis == 0 ? U : V, J = axis == 0 ? V : U;
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    double re = 0.0, im = 0.0;
    for (int j = 0; j < J; ++j) {
      double sn, cs;
      sincospi(2.0 * (j - J / 2) * frac, &sn, &cs);
      const cx<T> v = axis == 0 ? S[j * U + k] : S[k * U + j];
      re += (double)v.x * cs - (double)v.y * sn;
      im += (double)v.x * sn + (double)v.y * cs;
    }
    Tk[k] = {(T)re, (T)im};
  }
  __syncthreads();
  const int plane = pc / 3, comp = pc % 3;
  cx<T>* dst = E + ((long long)comp * fz + plane) * n;
  for (int f = threadIdx.x; f < n; f += blockDim.x) {
    const cx<T> w = tw[f], sh = tw[n + f];
    cx<T> acc = Tk[K - 1];
    for (int k = K - 2; k >= 0; --k) acc = cmuladd(acc, w, Tk[k]);
    dst[f] = cmul(acc, sh);
  }
}

// ---------------------------------------------------------------- objective, intensity
// An ideal objective's coherent transfer function on the per-plane spectra:
// modes whose direction sine exceeds the numerical aperture are removed.
template <typename T>
__global__ void objective_kernel(cx<T>* __restrict__ spec, long long n, int M, int U, int V,
                                 double sx_step, double sy_step, double na2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int m = (int)(i % M);
  const double sx = (m % U - U / 2) * sx_step, sy = (m / U - V / 2) * sy_step;
  if (sx * sx + sy * sy > na2) spec[i] = {0, 0};
}

// A general transfer function on the per-plane spectra: every mode's
// coefficients times H[m] (complex128, applied in FP64).
template <typename T>
__global__ void transfer_kernel(cx<T>* __restrict__ spec, long long n, int M,
                                const double2* __restrict__ H) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 h = H[i % M];
  const cx<T> v = spec[i];
  spec[i] = {(T)((double)v.x * h.x - (double)v.y * h.y), (T)((double)v.x * h.y + (double)v.y * h.x)};
}

template <typename T>
__global__ void intensity_kernel(const cx<T>* __restrict__ E, T* __restrict__ I, long long npix) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npix) return;
  const cx<T> a = E[i], b = E[npix + i], c = E[2 * npix + i];
  I[i] = a.x * a.x + a.y * a.y + b.x * b.x + b.y * b.y + c.x * c.x + c.y * c.y;
}

template <typename T>
hipError_t launch_idft_fft(const SynthArgs& a, hipStream_t s) {
  const int P = a.fft_p, R = a.fy / P;
  const int cols = a.idft_gtiles == 32 ? 32 : 64;  // columns per block
  const size_t lds = ((size_t)a.U * a.V + 32 * (size_t)cols + 32 * (size_t)R) * sizeof(cx<T>);
  dim3 grid((a.fx + cols - 1) / cols, a.fz * 3);
  const cx<T>* tw1 = reinterpret_cast<const cx<T>*>(a.fft_tw);
  auto go = [&](auto kern) {
    kern<<<grid, 256, lds, s>>>(reinterpret_cast<const cx<T>*>(a.spec),
                                reinterpret_cast<const cx<T>*>(a.twx), tw1, a.U, a.V, a.fx,
                                a.fy, a.fz, reinterpret_cast<cx<T>*>(a.E));
  };
  auto radix = [&](auto cols_tag) -> hipError_t {
    constexpr int C = decltype(cols_tag)::value;
    switch (P) {
      case 2: go(idft_fft_kernel<T, 2, C>); break;
      case 4: go(idft_fft_kernel<T, 4, C>); break;
      case 8: go(idft_fft_kernel<T, 8, C>); break;
      case 16: go(idft_fft_kernel<T, 16, C>); break;
      case 32: go(idft_fft_kernel<T, 32, C>); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  };
  return cols == 32 ? radix(std::integral_constant<int, 32>())
                    : radix(std::integral_constant<int, 64>());
}

template <typename T>
hipError_t launch_idft(const SynthArgs& a, hipStream_t s) {
  const int n_pc = a.fz * 3;
  auto go = [&](auto ft_tag) -> hipError_t {
    constexpr int FT = decltype(ft_tag)::value;
    const int nft = (a.fx + FT - 1) / FT;
    // enough g tiles for ~2 blocks per CU, but at least 64 rows per tile
    int ng = 1;
    while ((long long)n_pc * nft * ng < 512 && a.fy / (ng * 2) >= 64) ng *= 2;
    if (a.idft_gtiles > 0) ng = a.idft_gtiles;
    const int grows = (a.fy + ng - 1) / ng;
    const size_t lds = ((size_t)a.U * a.V + (size_t)a.V * FT) * sizeof(cx<T>);
    dim3 grid(nft, (a.fy + grows - 1) / grows, n_pc);
    idft_kernel<T, FT><<<grid, FT, lds, s>>>(
        reinterpret_cast<const cx<T>*>(a.spec), reinterpret_cast<const cx<T>*>(a.twx),
        reinterpret_cast<const cx<T>*>(a.twy), a.U, a.V, a.fx, a.fy, a.fz, grows,
        reinterpret_cast<cx<T>*>(a.E));
    return hipGetLastError();
  };
  if (a.fx <= 64) return go(std::integral_constant<int, 64>());
  if (a.fx <= 128) return go(std::integral_constant<int, 128>());
  return go(std::integral_constant<int, 256>());
}

inline unsigned blocks_for(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

template <typename T, int ZT>
hipError_t launch_modal(const SynthArgs& a, hipStream_t s, bool phases, const ExtArgs& x) {
  constexpr int RW = (sizeof(T) == 4) ? (ZT <= 4 ? 8 : 4) : (ZT <= 2 ? 4 : 2);
  const int n2 = 2 * a.M;
  const int rows_per_block = 4 * RW;
  const int nb_xy = (n2 + rows_per_block - 1) / rows_per_block;
  const int nb_z = (a.M + rows_per_block - 1) / rows_per_block;
  const size_t max_lds = 64 * 1024;
  int jc = (int)(max_lds / (ZT * sizeof(cx<T>)));
  jc = jc >= n2 ? n2 : (jc / 64) * 64;
  const size_t lds = (size_t)ZT * jc * sizeof(cx<T>);
  const long long nblocks = (long long)a.ntasks * (nb_xy + nb_z);
  if (nblocks == 0) return hipSuccess;
  auto go = [&](auto kern) {
    const long long ext = ((long long)x.n_ext * 3 * a.M + 255) / 256;
    kern<<<(unsigned)(nblocks + ext), 256, lds, s>>>(
        reinterpret_cast<const cx<T>*>(a.P), reinterpret_cast<const cx<T>*>(a.w),
        reinterpret_cast<const zd*>(a.kg), reinterpret_cast<const zd*>(a.a),
        reinterpret_cast<const zd*>(a.b), a.task_dz, a.tasks, a.M, nb_xy, nb_z, jc,
        (int)nblocks, x, reinterpret_cast<cx<T>*>(a.spec));
    return hipGetLastError();
  };
  return phases ? go(modal_kernel<T, ZT, RW, true>) : go(modal_kernel<T, ZT, RW, false>);
}

template <typename T>
hipError_t launch_synthesis(const SynthArgs& a, hipStream_t s, hipEvent_t* ev) {
  hipError_t e;
  const int n2 = 2 * a.M;
  auto mark = [&](int i) -> hipError_t { return ev ? hipEventRecord(ev[i], s) : hipSuccess; };
  if ((e = mark(0)) != hipSuccess) return e;
  const bool modal = (a.stages & kStageModal) != 0;
  const ExtArgs x{reinterpret_cast<const ExtPlane*>(a.ext_planes),
                  reinterpret_cast<const zd*>(a.ext), reinterpret_cast<const zd*>(a.ksz),
                  (a.stages & kStageExterior) ? a.n_ext : 0};
  // the exterior planes ride with the modal sum, unless the stages are timed
  const bool ride = modal && a.ntasks > 0 && a.nvol == 1 && !ev;
  ExtArgs xm = x;
  if (!ride) xm.n_ext = 0;
  if (!modal) {
    if ((e = mark(1)) != hipSuccess) return e;
  } else if (a.ntasks > 0) {
    if constexpr (sizeof(T) == 8) {
      // The phases of a task are made in the modal sum's blocks where a thread
      // makes at most six (each block repeats them), in a launch before it
      // otherwise. 4 tasks of 8 planes: M = 25 12.8 us a call fused, 18.2 with the
      // launch; M = 81 15.9 and 16.5; M = 121 16.9 and 16.5; 8 tasks at M = 225
      // 28.2 and 22.2.
      const bool fused = (long long)a.zt * n2 <= 1536;
      if (!fused) {
        phase_kernel<T><<<blocks_for((long long)a.ntasks * a.zt * n2, 256), 256, 0, s>>>(
            a.tasks, a.task_dz, reinterpret_cast<const zd*>(a.kg),
            reinterpret_cast<const zd*>(a.a), reinterpret_cast<const zd*>(a.b), n2, a.zt,
            a.ntasks, reinterpret_cast<cx<T>*>(a.w));
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      if ((e = mark(1)) != hipSuccess) return e;
      switch (a.zt) {
        case 1: e = launch_modal<T, 1>(a, s, fused, xm); break;
        case 2: e = launch_modal<T, 2>(a, s, fused, xm); break;
        case 4: e = launch_modal<T, 4>(a, s, fused, xm); break;
        case 8: e = launch_modal<T, 8>(a, s, fused, xm); break;
        default: return hipErrorInvalidValue;
      }
      if (e != hipSuccess) return e;
    } else {
      if ((e = mark(1)) != hipSuccess) return e;
      switch (a.zt) {
        case 1: e = launch_modal_f32<1>(a, s, xm); break;
        case 2: e = launch_modal_f32<2>(a, s, xm); break;
        case 4: e = launch_modal_f32<4>(a, s, xm); break;
        case 8: e = launch_modal_f32<8>(a, s, xm); break;
        default: return hipErrorInvalidValue;
      }
      if (e != hipSuccess) return e;
    }
  } else if ((e = mark(1)) != hipSuccess) {
    return e;
  }
  if ((e = mark(2)) != hipSuccess) return e;
  if (x.n_ext > 0 && !ride) {
    exterior_kernel<T><<<dim3(blocks_for((long long)x.n_ext * 3 * a.M, 256), a.nvol), 256, 0, s>>>(
        x, a.M, (long long)a.fz * 3 * a.M, reinterpret_cast<cx<T>*>(a.spec));
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = mark(3)) != hipSuccess) return e;
  if (!(a.stages & kStageTransform)) {
    // transform not requested
  } else if (a.pair_tab) {
    if ((e = launch_idft_pair(a, s)) != hipSuccess) return e;
  } else if (a.fft_p > 0) {
    if ((e = launch_idft_fft<T>(a, s)) != hipSuccess) return e;
  } else if (sizeof(T) == 4 && a.mfma) {
    MfmaArgs m{a.U, a.V, a.fx, a.fy, a.fz, a.kp, a.idft_gtiles, a.spec, a.twx, a.bmat, a.bscale, a.amat, a.E};
    if ((e = launch_idft_mfma(m, a.precision, s)) != hipSuccess) return e;
  } else if ((e = launch_idft<T>(a, s)) != hipSuccess) {
    return e;
  }
  return mark(4);
}

}  // namespace

hipError_t launch_modal_multi(const void* P, const void* kg, const void* ab, const Task* tasks,
                              const void* task_dz32, int ntasks, int zt, int M, int L, int fz,
                              int k0, int kcount, void* W, void* spec, hipStream_t s) {
  if (zt < 1 || zt > 8 || 32 % zt != 0 || kcount < 1 || kcount * zt > 32)
    return hipErrorInvalidValue;
  if (ntasks == 0) return hipSuccess;
  const int n2p = multi_row_pitch(M);
  multi_phase_kernel<<<blocks_for((long long)ntasks * 32 * n2p, 256), 256, 0, s>>>(
      reinterpret_cast<const float2*>(kg), reinterpret_cast<const float2*>(ab), tasks,
      reinterpret_cast<const float2*>(task_dz32), zt, M, L, n2p, k0, kcount, ntasks,
      reinterpret_cast<float2*>(W));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nb_xy = (2 * M + 15) / 16, nb_z = (M + 15) / 16;
  const long long nblocks = (long long)ntasks * (nb_xy + nb_z);
  modal_multi_kernel<<<(unsigned)((nblocks + 7) / 8 * 8), 256, 0, s>>>(
      reinterpret_cast<const float4*>(P), reinterpret_cast<const float4*>(W), tasks, zt, M, fz,
      n2p, k0, kcount, ntasks, nb_xy, nb_z, reinterpret_cast<float2*>(spec));
  return hipGetLastError();
}

hipError_t launch_synthesis_fp64(const SynthArgs& a, hipStream_t s, hipEvent_t* ev) {
  return launch_synthesis<double>(a, s, ev);
}
hipError_t launch_objective(void* spec, long long n, int M, int U, int V, double sx_step,
                            double sy_step, double na, bool fp64, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned nb = blocks_for(n, 256);
  if (fp64)
    objective_kernel<double><<<nb, 256, 0, s>>>(reinterpret_cast<cx<double>*>(spec), n, M, U, V,
                                                sx_step, sy_step, na * na);
  else
    objective_kernel<float><<<nb, 256, 0, s>>>(reinterpret_cast<cx<float>*>(spec), n, M, U, V,
                                               sx_step, sy_step, na * na);
  return hipGetLastError();
}

hipError_t launch_transfer(void* spec, long long n, int M, const void* H, bool fp64,
                           hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned nb = blocks_for(n, 256);
  const double2* h = reinterpret_cast<const double2*>(H);
  if (fp64)
    transfer_kernel<double><<<nb, 256, 0, s>>>(reinterpret_cast<cx<double>*>(spec), n, M, h);
  else
    transfer_kernel<float><<<nb, 256, 0, s>>>(reinterpret_cast<cx<float>*>(spec), n, M, h);
  return hipGetLastError();
}

hipError_t launch_intensity(const void* E, void* I, long long npix, bool fp64, hipStream_t s) {
  if (npix <= 0) return hipSuccess;
  const unsigned nb = blocks_for(npix, 256);
  if (fp64)
    intensity_kernel<double><<<nb, 256, 0, s>>>(reinterpret_cast<const cx<double>*>(E),
                                                reinterpret_cast<double*>(I), npix);
  else
    intensity_kernel<float><<<nb, 256, 0, s>>>(reinterpret_cast<const cx<float>*>(E),
                                               reinterpret_cast<float*>(I), npix);
  return hipGetLastError();
}

hipError_t launch_slice(const SliceArgs& a, bool fp64, hipStream_t s) {
  const int K = a.axis == 0 ? a.U : a.V;
  if (a.fz * 3 < 1) return hipSuccess;
  auto go = [&](auto tag) -> hipError_t {
    using T = decltype(tag);
    const size_t lds = ((size_t)a.U * a.V + K) * sizeof(cx<T>);
    slice_kernel<T><<<a.fz * 3, 256, lds, s>>>(
        reinterpret_cast<const cx<T>*>(a.spec), reinterpret_cast<const cx<T>*>(a.tw), a.U, a.V,
        a.n, a.fz, a.axis, a.frac, reinterpret_cast<cx<T>*>(a.E));
    return hipGetLastError();
  };
  return fp64 ? go(double{}) : go(float{});
}

// Copies a field [np][fy][fx] (np = 3 fz plane-components) into the window
// at (ox, oy) of a wider field [np][dfy][dfx], rx x ry times side by side.
template <typename T>
__global__ void place_kernel(const cx<T>* __restrict__ src, int fx, int fy, long long total,
                             cx<T>* __restrict__ dst, int dfx, int dfy, int ox, int oy, int rx,
                             int ry) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int f = (int)(i % fx);
  const long long q = i / fx;
  const int g = (int)(q % fy);
  const long long pc = q / fy;
  const cx<T> v = src[i];
  for (int ty = 0; ty < ry; ++ty) {
    cx<T>* row = dst + (pc * dfy + oy + (long long)ty * fy + g) * dfx + ox + f;
    for (int tx = 0; tx < rx; ++tx) row[(long long)tx * fx] = v;
  }
}

hipError_t launch_place(const void* src, int fx, int fy, int fz, void* dst, int dfx, int dfy,
                        int ox, int oy, int rx, int ry, bool fp64, hipStream_t s) {
  const long long total = 3LL * fz * fy * fx;
  if (total <= 0) return hipSuccess;
  const unsigned nb = blocks_for(total, 256);
  if (fp64)
    place_kernel<double><<<nb, 256, 0, s>>>(reinterpret_cast<const cx<double>*>(src), fx, fy,
                                            total, reinterpret_cast<cx<double>*>(dst), dfx, dfy,
                                            ox, oy, rx, ry);
  else
    place_kernel<float><<<nb, 256, 0, s>>>(reinterpret_cast<const cx<float>*>(src), fx, fy,
                                           total, reinterpret_cast<cx<float>*>(dst), dfx, dfy,
                                           ox, oy, rx, ry);
  return hipGetLastError();
}

hipError_t launch_synthesis_fp32(const SynthArgs& a, hipStream_t s, hipEvent_t* ev) {
  return launch_synthesis<float>(a, s, ev);
}

}  // namespace scw
