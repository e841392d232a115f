// Inverse transform of the plane spectra by conjugate pairs (Eq. 10), the
// library's choice for FP32 and FP64 grids with V <= 33:
//   E[g][f] = sum_{v,u} S[v][u] exp(2 pi i (u f / fx + v g / fy)),
// with u and v counted from -U/2 and -V/2, as a sum over u, then over v.
//
// Terms +-k of a sum have conjugate factors cos(t) +- i sin(t), so with
//   A = X_0 + sum_k cos(t_k) (X_k + X_-k),  B = i sum_k sin(t_k) (X_k - X_-k)
// the value at a point is A + B, and A - B at the point with -t. Let c be an
// axis' middle, (n - 1) / 2, and c +- d its points in pairs (d = 1/2, 3/2, ...
// for even n; 0, 1, 2, ... for odd n): with the phase of c folded into X, a pair
// takes 4 real multiply-adds per k, a quarter of the direct sum's, for any n.
// The y pass of an even axis halves that again: its rows d and n/2 - d have the
// same cosines and sines up to (-1)^k, so the sums over even and over odd k, once
// formed, give four rows. A point then costs about 11 multiply-adds at V = 21.
//
// Block = 32 pairs of columns of one plane/component, 256 threads. The
// spectrum's sums and differences over u and the pairs' factors go to LDS; x
// pass: a thread takes one pair and every eighth row v. y pass: a lane keeps its
// column's sums and differences over v in registers (lanes 0..31 the upper
// columns, 32..63 the lower ones, both in rising order) and every wave takes
// each fourth group of rows, whose factors are wave-uniform and come through the
// scalar cache: the loop is multiply-adds and stores alone. It is bound by the
// field's stores: 201 MB (256 x 256 x 128 points, U = V = 21) take 34.7 us (a
// fill of those bytes 29.7), or 44.3 past the cache (42.2). With rows in pairs
// only 47.7 past the cache, and one column per lane in the x pass 49.6.
//
// With NC = 3 a block takes the three components of a plane, keeps all three
// columns in registers and also writes |E_x|^2 + |E_y|^2 + |E_z|^2, which
// saves the pass that would read the field again.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "scw_internal.h"

namespace scw {
namespace {

template <typename T>
struct cx {
  T x, y;
};

template <typename T>
struct PairArgs {
  PairLayout lay;
  int U, V, fx, fy, fz, tiles, splits;
  int objective;
  double sx_step, sy_step, na2;
};

template <typename T>
__device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

template <bool NT, typename T>
__device__ __forceinline__ void store(T* d, T v) {
  if constexpr (NT)
    __builtin_nontemporal_store(v, d);
  else
    *d = v;
}
template <bool NT, typename T>
__device__ __forceinline__ void store(cx<T>* d, cx<T> v) {
  typedef T t2v __attribute__((ext_vector_type(2)));
  store<NT>(reinterpret_cast<t2v*>(d), t2v{v.x, v.y});
}

// Bytes of the last-level cache. A field that fits stays there when stored
// normally, which is the faster store (waves of 8 x 25 MB: 40.2 us, non-temporal
// 42.4). It evicts the synthesis matrix, though, and leaves lines to write back:
// with 300 MB of matrix and 201 MB of field the next modal sum takes 88 us
// against 56. So stores go past the cache where the field alone does not fit
// (369 MB: a pass of 116 us against 121), or where both do not and the matrix
// is of the field's order (44 MB and 236 MB: normal, 69 us against 77).
constexpr double kLastCache = 256.0 * 1024 * 1024;

// HV: pairs +-v kept in registers, V / 2 <= HV (the table is zero past V / 2).
// QUAD: fy is even, four rows to a group; else two.
// spec_all [vol][fz][3][V][U]; tab: pair_layout; E_all [vol][3][fz][fy][fx];
// I [fz][fy][fx] (NC = 3).
template <typename T, int HV, int NC, bool QUAD, bool NT>
__global__ void __launch_bounds__(256)
idft_pair_kernel(const PairArgs<T> a, cx<T>* spec_all, const cx<T>* __restrict__ tab,
                 cx<T>* __restrict__ E_all, T* __restrict__ I) {
  extern __shared__ unsigned char smem_raw[];
  const int U = a.U, V = a.V, HU = U / 2, M = U * V;
  struct Quad {
    cx<T> sum, diff;
  };
  Quad* Ss = reinterpret_cast<Quad*>(smem_raw);                 // [NC][V][HU + 1]
  cx<T>* cw = reinterpret_cast<cx<T>*>(Ss + NC * V * (HU + 1));  // [HU][32]
  cx<T>* Ts = cw + HU * 32;                                     // [NC][V][64]
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int tile = blockIdx.x % a.tiles, split = blockIdx.x / a.tiles;
  const int plane = NC == 3 ? blockIdx.y : blockIdx.y / 3;
  const int comp0 = NC == 3 ? 0 : blockIdx.y % 3;
  const long long vol = blockIdx.z;
  const cx<T>* xph = tab + a.lay.xph;
  cx<T>* spec = spec_all + ((vol * a.fz + plane) * 3 + comp0) * M;
  for (int i = t; i < NC * V * (HU + 1); i += 256) {
    const int u = i % (HU + 1), cv = i / (HU + 1), v = cv % V;
    const long long o = (long long)cv * U + HU;  // (component, v) rows of U
    cx<T> p = spec[o + u], q = spec[o - u];
    if (a.objective) {  // modes beyond the aperture are removed
      const double sx = u * a.sx_step, sy = (v - V / 2) * a.sy_step;
      if (sx * sx + sy * sy > a.na2) {
        p = q = {0, 0};
        if (tile == 0 && split == 0) spec[o + u] = spec[o - u] = {0, 0};
      }
    }
    const cx<T> w = xph[u];
    p = cmul(p, w);
    q = cmul(q, cx<T>{w.x, -w.y});
    Ss[i] = u == 0 ? Quad{p, {0, 0}} : Quad{{p.x + q.x, p.y + q.y}, {p.x - q.x, p.y - q.y}};
  }
  const int npx = a.lay.npx, p0 = tile * 32;
  for (int i = t; i < HU * 32; i += 256)
    cw[i] = tab[(long long)(i / 32) * npx + min(p0 + (i & 31), npx - 1)];
  __syncthreads();
  {
    const cx<T>* yph = tab + a.lay.yph;
    const int pl = t & 31;
    for (int cv = t >> 5; cv < NC * V; cv += 8) {
      const Quad* s = Ss + cv * (HU + 1);
      cx<T> A = s[0].sum, B = {0, 0};
#pragma unroll 5
      for (int u = 1; u <= HU; ++u) {
        const cx<T> w = cw[(u - 1) * 32 + pl];
        const Quad q = s[u];
        A.x = fma(w.x, q.sum.x, A.x);
        A.y = fma(w.x, q.sum.y, A.y);
        B.x = fma(-w.y, q.diff.y, B.x);
        B.y = fma(w.y, q.diff.x, B.y);
      }
      const cx<T> ph = yph[cv % V];
      Ts[cv * 64 + pl] = cmul(cx<T>{A.x + B.x, A.y + B.y}, ph);
      Ts[cv * 64 + 63 - pl] = cmul(cx<T>{A.x - B.x, A.y - B.y}, ph);
    }
  }
  __syncthreads();
  cx<T> mid[NC], sum[NC][HV], diff[NC][HV];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const cx<T>* col = Ts + (c * V + V / 2) * 64 + lane;
    mid[c] = col[0];
#pragma unroll
    for (int k = 0; k < HV; ++k) {
      const int v = min(k + 1, V / 2) * 64;
      const cx<T> p = col[v], q = col[-v];
      sum[c][k] = {p.x + q.x, p.y + q.y};
      diff[c][k] = {p.x - q.x, p.y - q.y};
    }
  }
  const int ex = 1 - (a.fx & 1), pair = p0 + (lane < 32 ? lane : 63 - lane);
  const int f = lane < 32 ? (a.fx - 1) / 2 + ex + pair : (a.fx - 1) / 2 - pair;
  if (pair >= npx || (lane >= 32 && !ex && pair == 0)) return;  // no barrier follows
  const int groups = a.lay.npy;
  const int j0 = (int)((long long)groups * split / a.splits);
  const int j1 = (int)((long long)groups * (split + 1) / a.splits);
  const long long fsize = (long long)a.fy * a.fx, vsize = fsize * a.fz;
  cx<T>* dst = E_all + (vol * 3 + comp0) * vsize + plane * fsize + f;
  T* idst = NC == 3 ? I + plane * fsize + f : nullptr;
  constexpr int R = QUAD ? 4 : 2;
  for (int j = j0 + wave; j < j1; j += 4) {
    const cx<T>* w = tab + a.lay.yw + (long long)j * HV;  // wave-uniform
    // the group's rows; the middle one of an odd axis, and the middle two of the
    // pairs where their number is odd, are met twice
    const int row[4] = {a.fy / 2 + j, (a.fy - 1) / 2 - j, a.fy - 1 - j, j};
    const int n = QUAD ? (row[0] < row[2] ? 4 : 2) : (j > 0 ? 2 : 1);
    T ir[R] = {};
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      cx<T> Ae = mid[c], Be = {0, 0}, Ao = {0, 0}, Bo = {0, 0};
#pragma unroll
      for (int k = 0; k < HV; ++k) {
        const cx<T> q = w[k];
        cx<T>& A = QUAD && k % 2 == 0 ? Ao : Ae;
        cx<T>& B = QUAD && k % 2 == 0 ? Bo : Be;
        A.x = fma(q.x, sum[c][k].x, A.x);
        A.y = fma(q.x, sum[c][k].y, A.y);
        B.x = fma(-q.y, diff[c][k].y, B.x);
        B.y = fma(q.y, diff[c][k].x, B.y);
      }
      cx<T> val[R];  // rows c + d, c - d, then c + n/2 - d, c - n/2 + d
      const cx<T> A = {Ae.x + Ao.x, Ae.y + Ao.y}, B = {Be.x + Bo.x, Be.y + Bo.y};
      val[0] = {A.x + B.x, A.y + B.y};
      val[1] = {A.x - B.x, A.y - B.y};
      if (QUAD) {
        const cx<T> C = {Ae.x - Ao.x, Ae.y - Ao.y}, D = {Be.x - Bo.x, Be.y - Bo.y};
        val[R - 2] = {C.x - D.x, C.y - D.y};
        val[R - 1] = {C.x + D.x, C.y + D.y};
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r < n) store<NT>(dst + c * vsize + (long long)row[r] * a.fx, val[r]);
        if (NC == 3) ir[r] += val[r].x * val[r].x + val[r].y * val[r].y;
      }
    }
    if (NC == 3) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r < n) store<NT>(idst + (long long)row[r] * a.fx, ir[r]);
    }
  }
}

template <typename T, int NC>
hipError_t launch(const SynthArgs& s, hipStream_t st) {
  PairArgs<T> a{};
  a.lay = pair_layout(s.U, s.V, s.fx, s.fy);
  a.U = s.U;
  a.V = s.V;
  a.fx = s.fx;
  a.fy = s.fy;
  a.fz = s.fz;
  a.tiles = (a.lay.npx + 31) / 32;
  const double field = (double)s.nvol * 3 * s.fz * s.fy * s.fx * sizeof(cx<T>);
  const double matrix = (double)s.L * 6 * s.M * s.M * sizeof(cx<T>);
  const bool nt = field > kLastCache || (field + matrix > kLastCache && 2 * matrix > field);
  a.objective = s.objective;
  a.sx_step = s.sx_step;
  a.sy_step = s.sy_step;
  a.na2 = s.na2;
  const size_t lds = ((size_t)NC * s.V * (s.U / 2 + 1) * 2 + (size_t)(s.U / 2) * 32 +
                      (size_t)NC * s.V * 64) * sizeof(cx<T>);
  // rows split over blocks while the launch has less than two blocks per CU, each
  // wave keeps four groups of rows and the blocks stay one round by their LDS (a
  // split repeats the x pass: 128 x 128 x 64 in FP64 at V = 31, two blocks to a
  // CU, 20.2 us whole, 25.9 split)
  const long long blocks = (long long)a.tiles * (NC == 3 ? 1 : 3) * s.fz * s.nvol;
  const long long slots = 256 * std::max<long long>(1, 160 * 1024 / (long long)std::max<size_t>(lds, 1));
  a.splits = 1;
  while (blocks * a.splits < 512 && blocks * a.splits * 2 <= slots &&
         a.lay.npy / (a.splits * 2) >= 16)
    a.splits *= 2;
  const dim3 grid(a.tiles * a.splits, (NC == 3 ? 1 : 3) * s.fz, s.nvol);
  auto go = [&](auto kern) {
    kern<<<grid, 256, lds, st>>>(a, reinterpret_cast<cx<T>*>(s.spec),
                                 reinterpret_cast<const cx<T>*>(s.pair_tab),
                                 reinterpret_cast<cx<T>*>(s.E), reinterpret_cast<T*>(s.I));
    return hipGetLastError();
  };
  auto pick = [&](auto quad, auto through) {
    constexpr bool Q = decltype(quad)::value, S = decltype(through)::value;
    switch (a.lay.hv) {
      case 2: return go(idft_pair_kernel<T, 2, NC, Q, S>);
      case 4: return go(idft_pair_kernel<T, 4, NC, Q, S>);
      case 6: return go(idft_pair_kernel<T, 6, NC, Q, S>);
      case 8: return go(idft_pair_kernel<T, 8, NC, Q, S>);
      case 10: return go(idft_pair_kernel<T, 10, NC, Q, S>);
      case 12: return go(idft_pair_kernel<T, 12, NC, Q, S>);
      case 16: return go(idft_pair_kernel<T, 16, NC, Q, S>);
      default: return hipErrorInvalidValue;
    }
  };
  const std::true_type yes;
  const std::false_type no;
  if (s.fy % 2) return nt ? pick(no, yes) : pick(no, no);
  return nt ? pick(yes, yes) : pick(yes, no);
}

}  // namespace

// Tables of idft_pair_kernel, in complex values: the column pairs' factors (cos,
// sin) [u = 1 .. U/2][pair], the phases of the middle column for u = 0 .. U/2,
// the row groups' factors [group][hv] for v = 1 .. hv (zero past V/2), and the
// phases of the middle row for v = -V/2 .. V/2.
PairLayout pair_layout(int U, int V, int fx, int fy) {
  PairLayout l{};
  const int h = V / 2;
  l.hv = h <= 2 ? 2 : h <= 4 ? 4 : h <= 6 ? 6 : h <= 8 ? 8 : h <= 10 ? 10 : h <= 12 ? 12 : 16;
  l.npx = (fx + 1) / 2;
  l.npy = fy % 2 ? (fy + 1) / 2 : (fy / 2 + 1) / 2;
  l.xph = (long long)(U / 2) * l.npx;
  l.yw = l.xph + U / 2 + 1;
  l.yph = l.yw + (long long)l.npy * l.hv;
  l.size = l.yph + V;
  return l;
}

// The kernel's LDS (64 KB at most): one component, or the three of a plane.
bool pair_transform_fits(int U, int V, bool fp64, int components) {
  return V <= 33 && ((size_t)components * V * (U / 2 + 1) * 2 + (size_t)(U / 2) * 32 +
                     (size_t)components * V * 64) * (fp64 ? 16 : 8) <= 64 * 1024;
}

hipError_t launch_idft_pair(const SynthArgs& a, hipStream_t s) {
  if (a.precision == SCW_FP64) return a.I ? hipErrorInvalidValue : launch<double, 1>(a, s);
  return a.I ? launch<float, 3>(a, s) : launch<float, 1>(a, s);
}

}  // namespace scw
