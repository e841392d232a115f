// Batched FP64 complex non-symmetric eigensolver for the per-layer 2M x 2M
// products A C (Sec. 3.2, Sec. 4.2: the eigendecomposition step). Every
// matrix of a batch is independent: the two chains of dependent steps (the
// reduction's panels and the QR iteration) have one workgroup per matrix, so
// that a batch of layers, wavelengths or patches fills the chip; what the chains
// leave behind (their reflectors and rotations on the rest of H and on Z, and the
// eigenvectors) is spread over many workgroups to a matrix.
//
// Steps, each a published method restated for this layout:
//   1. Householder reduction to upper Hessenberg form H = Q^H A Q in panels of
//      reflectors, which are then accumulated into Z = Q (Golub & Van Loan,
//      Matrix Computations, Sec. 7.4; the compact form Q = I - V T V^H of
//      Schreiber and Van Loan).
//   2. Complex Schur form T = Z^H A Z by the implicitly shifted single-shift
//      QR algorithm on H: Wilkinson shifts with exceptional shifts after 10
//      and 20 stalled iterations, deflation on negligible subdiagonals
//      (Golub & Van Loan, Sec. 7.5; the complex form of LAPACK's xLAHQR). The
//      iteration works on the active diagonal block; its rotations are
//      recorded and then applied to the rest of H and to Z.
//   3. Eigenvectors of T by back-substitution, (T - t_jj I) y_j = 0 with
//      y_j(j) = 1, perturbing a vanishing pivot to eps |t_jj| as xTREVC does.
//      The eigenvectors of A are Z y_j (a batched matrix product done by the
//      caller), normalised to unit length.
// All matrices are column-major, complex128, n x n, stored one after another.
#include <hip/hip_runtime.h>

#include <cfloat>

#include "scw_internal.h"

namespace scw {
namespace {

constexpr int kMaxSweepsPerEigenvalue = 300;
constexpr int kEigWindow = 16;  // rotations per window of the QR sweep (20 and 24 spill registers: 1.15x)
constexpr int kEigInner = 64;   // active blocks up to this order stay in LDS

__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// conj(a) * b
__device__ inline double2 cmulcj(double2 a, double2 b) {
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ inline double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
__device__ inline double cabs1(double2 a) { return fabs(a.x) + fabs(a.y); }
__device__ inline double cabs(double2 a) { return hypot(a.x, a.y); }

// a / b by Smith's method (no overflow for moderate ratios).
__device__ inline double2 cdiv(double2 a, double2 b) {
  if (fabs(b.x) >= fabs(b.y)) {
    const double r = b.y / b.x, den = b.x + b.y * r;
    return make_double2((a.x + a.y * r) / den, (a.y - a.x * r) / den);
  }
  const double r = b.x / b.y, den = b.x * r + b.y;
  return make_double2((a.x * r + a.y) / den, (a.y * r - a.x) / den);
}

// Principal square root (Re >= 0).
__device__ inline double2 csqrt(double2 z) {
  const double m = cabs(z);
  if (m == 0.0) return make_double2(0.0, 0.0);
  const double re = sqrt(0.5 * (m + fabs(z.x)));
  const double im = z.y / (2.0 * re);
  if (z.x >= 0.0) return make_double2(re, im);
  return make_double2(fabs(im), copysign(re, z.y));
}

__device__ inline double2 shfl_xor2(double2 v, int mask) {
  return make_double2(__shfl_xor(v.x, mask, 64), __shfl_xor(v.y, mask, 64));
}
__device__ inline double2 wave_sum(double2 v) {
  for (int m = 32; m >= 1; m >>= 1) v = cadd(v, shfl_xor2(v, m));
  return v;
}

typedef double dx4 __attribute__((ext_vector_type(4)));
// D += A B on 16 x 16 x 4 (v_mfma_f64_16x16x4_f64): lane l holds A[l % 16][l / 16]
// and B[l / 16][l % 16]; entry i of lane l is D[4 i + l / 16][l % 16].
__device__ inline dx4 mm4(double a, double b, dx4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Step 1. Householder reduction in panels of kPanel columns (the blocked form of
// LAPACK's xGEHRD / xLAHR2). With the panel's reflectors Q = I - V T V^H
// (T upper triangular), the rows k0 + 1 .. n - 1 of the columns right of the
// panel become
//   C <- (I - V T^H V^H) (C - Y V^H),   Y = A V T,
// where A V needs only the trailing matrix as it was before the panel: one
// reading per column (the product with the newest reflector), instead of six
// and three writings of H and Q when each reflector was applied at once.
// Rows 0 .. k0 of H and all of Q see the panel only from the right, row by row;
// eig_hess_apply_kernel does them afterwards, many workgroups to a matrix.
//
// One workgroup of 16 waves per matrix. Per column: update it by the panel so
// far (a thread per row), V^H a (a wave per reflector), the reflector, then
// A v with the rows over the threads and the columns over what groups of
// threads are left. The trailing update runs on the matrix cores in 16 x 16
// tiles. The reflectors are left below H's subdiagonal (with their leading 1
// implied) for the second kernel, which clears them, the T factors in Tall.
//
// 96 matrices of order 242: 46.2 ms with unblocked reflections (20 GB/s per
// workgroup).
constexpr int kPanel = 16;
// Workspace per matrix, in complex values: V, Y, W (kPanel x n each, column
// major, ld n) and the T factors of ceil(n / kPanel) panels.
__host__ __device__ inline size_t hess_work(int n) {
  return (size_t)3 * kPanel * n + (size_t)((n + kPanel - 1) / kPanel) * kPanel * kPanel;
}
__global__ void __launch_bounds__(1024)
eig_hessenberg_kernel(int n, double2* __restrict__ Aall, double2* __restrict__ work) {
  constexpr int NB = kPanel;
  extern __shared__ double2 lds[];  // acol [n], part [1024]
  double2* acol = lds;
  double2* part = lds + n;
  __shared__ double2 s_T[NB][NB];  // T[p][q]
  __shared__ double2 s_S[NB][NB];  // V^H Y, then T^H V^H Y
  __shared__ double2 s_row[NB], s_w[NB], s_u[NB];
  __shared__ double s_red[16];
  double2* A = Aall + (size_t)blockIdx.x * n * n;
  double2* V = work + (size_t)blockIdx.x * hess_work(n);
  double2* Y = V + (size_t)NB * n;
  double2* Wb = Y + (size_t)NB * n;
  double2* Tg = Wb + (size_t)NB * n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double2 zero = make_double2(0.0, 0.0);
  const int nref = n - 2;  // reflectors, one per column 0 .. n - 3
  for (int k0 = 0; k0 < nref; k0 += NB) {
    const int jn = min(NB, nref - k0), r0 = k0 + 1, m = n - r0;
    // A v: rows over rt threads, columns over ng groups of them
    const int rt = min(1024, (m + 63) / 64 * 64), ng = 1024 / rt;
    const int grp = tid / rt, rid = tid - grp * rt;
    if (tid < NB * NB) {
      s_T[tid / NB][tid % NB] = zero;
      s_S[tid / NB][tid % NB] = zero;
    }
    for (int q = jn; q < NB; ++q)  // a short panel ends in empty columns
      for (int r = r0 + tid; r < n; r += 1024) V[(size_t)q * n + r] = Y[(size_t)q * n + r] = zero;
    for (int j = 0; j < jn; ++j) {
      const int c = k0 + j;
      double2* ac = A + (size_t)c * n;
      // column c by the panel so far, from the right: - Y V[c, :]^H
      if (tid < j) s_row[tid] = cconj(V[(size_t)tid * n + c]);
      __syncthreads();
      for (int r = r0 + tid; r < n; r += 1024) {
        double2 a = ac[r];
        for (int q = 0; q < j; ++q) a = csub(a, cmul(Y[(size_t)q * n + r], s_row[q]));
        acol[r] = a;
      }
      __syncthreads();
      // and from the left: - V T^H (V^H a)
      if (wave < j) {
        double2 acc = zero;
        for (int r = r0 + lane; r < n; r += 64)
          acc = cadd(acc, cmulcj(V[(size_t)wave * n + r], acol[r]));
        acc = wave_sum(acc);
        if (lane == 0) s_w[wave] = acc;
      }
      __syncthreads();
      if (tid < j) {
        double2 acc = zero;
        for (int p = 0; p <= tid; ++p) acc = cadd(acc, cmulcj(s_T[p][tid], s_w[p]));
        s_u[tid] = acc;
      }
      __syncthreads();
      double norm2 = 0.0;
      for (int r = r0 + tid; r < n; r += 1024) {
        double2 a = acol[r];
        for (int q = 0; q < j; ++q) a = csub(a, cmul(V[(size_t)q * n + r], s_u[q]));
        acol[r] = a;
        if (r > c + 1) norm2 += a.x * a.x + a.y * a.y;
      }
      for (int o = 32; o >= 1; o >>= 1) norm2 += __shfl_xor(norm2, o, 64);
      if (lane == 0) s_red[wave] = norm2;
      __syncthreads();
      // the reflector: beta = -sign(Re alpha) ||(alpha, x)||, tau = (beta - alpha)
      // / beta, v = [1; x / (alpha - beta)]: (I - tau v v^H)^H [alpha; x] = [beta; 0]
      double x2 = 0.0;
#pragma unroll
      for (int q = 0; q < 16; ++q) x2 += s_red[q];
      const double2 alpha = acol[c + 1];
      double beta = alpha.x;
      double2 tau = zero, scale = zero;
      if (x2 != 0.0 || alpha.y != 0.0) {
        beta = -copysign(sqrt(alpha.x * alpha.x + alpha.y * alpha.y + x2), alpha.x);
        tau = make_double2((beta - alpha.x) / beta, -alpha.y / beta);
        scale = cdiv(make_double2(1.0, 0.0), make_double2(alpha.x - beta, alpha.y));
      }
      __syncthreads();  // every thread has read alpha
      for (int r = r0 + tid; r < n; r += 1024) {
        const double2 a = acol[r];
        const double2 v = r > c + 1 ? cmul(a, scale) : make_double2(r == c + 1 ? 1.0 : 0.0, 0.0);
        ac[r] = r > c + 1 ? v : (r == c + 1 ? make_double2(beta, 0.0) : a);
        acol[r] = v;
        V[(size_t)j * n + r] = v;
      }
      __syncthreads();
      // u = V^H v over the earlier reflectors, and A v in parts
      if (wave < j) {
        double2 acc = zero;
        for (int r = c + 1 + lane; r < n; r += 64)
          acc = cadd(acc, cmulcj(V[(size_t)wave * n + r], acol[r]));
        acc = wave_sum(acc);
        if (lane == 0) s_w[wave] = acc;
      }
      for (int rb = 0; rb < m; rb += rt) {
        const int r = min(r0 + rb + rid, n - 1);
        double2 acc = zero, acc2 = zero;
        if (grp < ng) {
          const double2* ap = A + r;
          int cc = c + 1 + grp;
          for (; cc + 7 * ng < n; cc += 8 * ng) {
            double2 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = ap[(size_t)(cc + u * ng) * n];
#pragma unroll
            for (int u = 0; u < 8; u += 2) {
              acc = cadd(acc, cmul(x[u], acol[cc + u * ng]));
              acc2 = cadd(acc2, cmul(x[u + 1], acol[cc + (u + 1) * ng]));
            }
          }
          for (; cc < n; cc += ng) acc = cadd(acc, cmul(ap[(size_t)cc * n], acol[cc]));
        }
        part[tid] = cadd(acc, acc2);
        __syncthreads();
        if (tid < rt && r0 + rb + tid < n) {
          double2 y = part[tid];
          for (int g = 1; g < ng; ++g) y = cadd(y, part[g * rt + tid]);
          for (int q = 0; q < j; ++q) y = csub(y, cmul(Y[(size_t)q * n + r0 + rb + tid], s_w[q]));
          Y[(size_t)j * n + r0 + rb + tid] = cmul(y, tau);
        }
        __syncthreads();
      }
      // T[:, j] = -tau T u, T[j][j] = tau
      if (tid <= j) {
        double2 t = zero;
        for (int q = tid; q < j; ++q) t = cadd(t, cmul(s_T[tid][q], s_w[q]));
        t = cmul(make_double2(-t.x, -t.y), tau);
        s_T[tid][j] = tid == j ? tau : t;
      }
      __syncthreads();
    }
    if (tid < NB * NB) Tg[(size_t)(k0 / NB) * NB * NB + tid] = s_T[tid / NB][tid % NB];
    // ---- the columns right of the panel
    const int c1 = k0 + jn, mc = n - c1;
    {  // S = V^H Y, a wave per row
      double2 acc[NB];
#pragma unroll
      for (int p = 0; p < NB; ++p) acc[p] = zero;
      for (int r = r0 + lane; r < n; r += 64) {
        const double2 v = V[(size_t)wave * n + r];
#pragma unroll
        for (int p = 0; p < NB; ++p) acc[p] = cadd(acc[p], cmulcj(v, Y[(size_t)p * n + r]));
      }
#pragma unroll
      for (int p = 0; p < NB; ++p) {
        const double2 t = wave_sum(acc[p]);
        if (lane == 0) s_S[wave][p] = t;
      }
    }
    const int lr = lane & 15, lk = lane >> 4;
    // W0 = V^H C: 16 x 16 tiles, K = the rows, four consecutive ones per lane
    for (int ct = wave * 16; ct < mc; ct += 256) {
      const int cc = min(c1 + ct + lr, n - 1);
      const double2* cp = A + (size_t)cc * n;
      const double2* vp = V + (size_t)lr * n;
      dx4 wr = {0.0, 0.0, 0.0, 0.0}, wi = wr;
#pragma unroll 2
      for (int rb = r0; rb < n; rb += 16) {
        double2 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = rb + 4 * lk + u, rc = min(r, n - 1);
          a[u] = vp[rc];
          b[u] = cp[rc];
          if (r >= n) a[u] = zero;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // conj(V) C
          wr = mm4(a[u].x, b[u].x, wr);
          wr = mm4(a[u].y, b[u].y, wr);
          wi = mm4(a[u].x, b[u].y, wi);
          wi = mm4(-a[u].y, b[u].x, wi);
        }
      }
      if (c1 + ct + lr < n)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          Wb[(size_t)(4 * u + lk) * n + c1 + ct + lr] = make_double2(wr[u], wi[u]);
    }
    __syncthreads();
    // W = T^H (W0 - S V[c, :]^H), a thread per column and four of its rows
    for (int e = tid; e < 4 * mc; e += 1024) {
      const int c = c1 + e / 4, q0 = (e % 4) * 4;
      double2 w[NB];
#pragma unroll
      for (int p = 0; p < NB; ++p) w[p] = Wb[(size_t)p * n + c];
#pragma unroll 1
      for (int q = 0; q < jn; ++q) {
        const double2 vc = cconj(V[(size_t)q * n + c]);
#pragma unroll
        for (int p = 0; p < NB; ++p) w[p] = csub(w[p], cmul(s_S[p][q], vc));
      }
      double2 o[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        o[u] = zero;
#pragma unroll
        for (int p = 0; p < NB; ++p) o[u] = cadd(o[u], cmulcj(s_T[p][q0 + u], w[p]));
      }
      // the four threads of a column are neighbours in one wave: all have read
      // W0 before any writes
#pragma unroll
      for (int u = 0; u < 4; ++u) Wb[(size_t)(q0 + u) * n + c] = o[u];
    }
    __syncthreads();
    // C -= Y V[c, :]^H + V W: tiles of 16 x 16, a wave per strip of rows
    const int tr = (m + 15) / 16, tc = (mc + 15) / 16;
    const int strips = min(16, tr), share = 16 / strips;  // waves per strip of rows
    for (int t = wave / share; t < tr; t += strips) {
      if (wave / share >= strips) break;
      const int rr = r0 + 16 * t;
      double2 ya[4], va[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = min(rr + lr, n - 1);
        ya[s] = Y[(size_t)(4 * s + lk) * n + r];
        va[s] = V[(size_t)(4 * s + lk) * n + r];
      }
      for (int u = wave % share; u < tc; u += share) {
        const int c = c1 + 16 * u + lr, cl = min(c, n - 1);
        dx4 cr, ci;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double2 x = A[(size_t)cl * n + min(rr + 4 * i + lk, n - 1)];
          cr[i] = x.x;
          ci[i] = x.y;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double2 vb = V[(size_t)(4 * s + lk) * n + cl];
          const double2 wb = Wb[(size_t)(4 * s + lk) * n + cl];
          // - Y conj(V)
          cr = mm4(-ya[s].x, vb.x, cr);
          cr = mm4(-ya[s].y, vb.y, cr);
          ci = mm4(ya[s].x, vb.y, ci);
          ci = mm4(-ya[s].y, vb.x, ci);
          // - V W
          cr = mm4(-va[s].x, wb.x, cr);
          cr = mm4(va[s].y, wb.y, cr);
          ci = mm4(-va[s].x, wb.y, ci);
          ci = mm4(-va[s].y, wb.x, ci);
        }
        if (c < n)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (rr + 4 * i + lk < n)
              A[(size_t)c * n + rr + 4 * i + lk] = make_double2(cr[i], ci[i]);
      }
    }
    __syncthreads();
  }
}

// The panels from the right, x <- x - ((x V) T) V^H, on the rows of Q (from the
// identity; z = 0) and on the rows of H that a panel's columns had left behind
// (row r <= k0; z = 1). A workgroup takes 64 rows, a lane each, its four waves
// a quarter of the columns each; V comes through LDS in chunks of 64 columns.
__global__ void __launch_bounds__(256)
eig_hess_apply_kernel(int n, double2* __restrict__ Hall, double2* __restrict__ Zall,
                      const double2* __restrict__ work) {
  constexpr int NB = kPanel, CH = 64;
  __shared__ double2 s_V[CH][NB];
  __shared__ double2 s_T[NB][NB];
  __shared__ double2 s_w[4][NB][64];
  const bool q_rows = blockIdx.z == 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int first = blockIdx.x * 64, row = first + lane;
  const double2* H = Hall + (size_t)blockIdx.y * n * n;
  double2* X = (q_rows ? Zall : Hall) + (size_t)blockIdx.y * n * n + min(row, n - 1);
  const double2* Tg = work + (size_t)blockIdx.y * hess_work(n) + (size_t)3 * NB * n;
  const double2 zero = make_double2(0.0, 0.0);
  if (q_rows && row < n)
    for (int c = wave; c < n; c += 4) X[(size_t)c * n] = make_double2(c == row ? 1.0 : 0.0, 0.0);
  const int nref = n - 2;
  for (int k0 = 0; k0 < nref; k0 += NB) {
    const int jn = min(NB, nref - k0);
    if (!q_rows && first > k0) continue;
    const bool on = row < n && (q_rows || row <= k0);
    __syncthreads();
    s_T[tid / NB][tid % NB] = Tg[(size_t)(k0 / NB) * NB * NB + tid];
    auto stage = [&](int c0) {  // V[c0 .. c0 + 63][:]
#pragma unroll
      for (int q = 0; q < CH * NB / 256; ++q) {
        const int e = tid + 256 * q, c = c0 + (e & 63), j = e >> 6, lead = k0 + j + 1;
        double2 v = zero;
        if (j < jn && c < n) {
          if (c > lead) v = H[(size_t)(k0 + j) * n + c];
          else if (c == lead) v = make_double2(1.0, 0.0);
        }
        s_V[e & 63][j] = v;
      }
    };
    double wx[NB], wy[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) wx[j] = wy[j] = 0.0;
    for (int c0 = k0 + 1; c0 < n; c0 += CH) {
      __syncthreads();
      stage(c0);
      __syncthreads();
#pragma unroll 4
      for (int i = 0; i < CH / 4; ++i) {
        const int cl = 4 * i + wave, c = c0 + cl;
        if (c >= n) break;
        const double2 x = X[(size_t)c * n];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const double2 v = s_V[cl][j];
          wx[j] += x.x * v.x - x.y * v.y;
          wy[j] += x.x * v.y + x.y * v.x;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) s_w[wave][j][lane] = make_double2(wx[j], wy[j]);
    __syncthreads();
    // w = (x V) T: the four partial sums, then the triangular factor
    double ux[NB], uy[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const double2 a = cadd(cadd(s_w[0][j][lane], s_w[1][j][lane]),
                             cadd(s_w[2][j][lane], s_w[3][j][lane]));
      wx[j] = a.x;
      wy[j] = a.y;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      ux[j] = uy[j] = 0.0;
#pragma unroll
      for (int p = 0; p <= j; ++p) {
        const double2 t = s_T[p][j];
        ux[j] += wx[p] * t.x - wy[p] * t.y;
        uy[j] += wx[p] * t.y + wy[p] * t.x;
      }
    }
    for (int c0 = k0 + 1; c0 < n; c0 += CH) {
      __syncthreads();
      stage(c0);
      __syncthreads();
#pragma unroll 4
      for (int i = 0; i < CH / 4; ++i) {
        const int cl = 4 * i + wave, c = c0 + cl;
        if (c >= n) break;
        double2 x = X[(size_t)c * n];
#pragma unroll
        for (int j = 0; j < NB; ++j) {  // - w conj(V)
          const double2 v = s_V[cl][j];
          x.x -= ux[j] * v.x + uy[j] * v.y;
          x.y -= uy[j] * v.x - ux[j] * v.y;
        }
        if (on) X[(size_t)c * n] = x;
      }
    }
  }
}

// Zeros below the subdiagonal, where the reflectors were.
__global__ void __launch_bounds__(256) eig_hess_clear_kernel(int n, double2* __restrict__ Hall) {
  double2* H = Hall + (size_t)blockIdx.y * n * n;
  const int c = blockIdx.x;
  for (int r = c + 2 + threadIdx.x; r < n; r += 256) H[(size_t)c * n + r] = make_double2(0.0, 0.0);
}

// Rotation G = [[c, s], [-conj(s), c]] with G [x; y] = [r; 0], c real.
__device__ inline void givens_scaled(double2 x, double2 y, double& c, double2& s,
                                           double2& r) {
  const double ax = cabs(x), ay = cabs(y);
  if (ay == 0.0) {
    c = 1.0;
    s = make_double2(0.0, 0.0);
    r = x;
    return;
  }
  if (ax == 0.0) {
    c = 0.0;
    s = cscale(cconj(y), 1.0 / ay);
    r = make_double2(ay, 0.0);
    return;
  }
  const double nrm = hypot(ax, ay);
  const double2 ph = cscale(x, 1.0 / ax);  // x / |x|
  c = ax / nrm;
  s = cscale(cmul(ph, cconj(y)), 1.0 / nrm);
  r = cscale(ph, nrm);
}
// 1 / sqrt(x) of a normal x: the hardware's estimate and one third-order step.
__device__ inline double rsqrt_normal(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
// The same from two reciprocal square roots where no square leaves the normal
// range (the chase waits for this result at every rotation).
__device__ inline void givens(double2 x, double2 y, double& c, double2& s, double2& r) {
  const double ax2 = x.x * x.x + x.y * x.y, ay2 = y.x * y.x + y.y * y.y, n2 = ax2 + ay2;
  const double rx = rsqrt_normal(ax2), rn = rsqrt_normal(n2), f = rx * rn;
  c = ax2 * f;
  s = cscale(cmul(x, cconj(y)), f);
  r = cscale(x, n2 * f);
  if (!(fmin(ax2, ay2) > 1e-250 && n2 < 1e250)) givens_scaled(x, y, c, s, r);
}

__device__ inline double2& at(double2* M, int n, int i, int j) { return M[(size_t)j * n + i]; }

__device__ inline double read_lane(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}
__device__ inline double2 read_lane(double2 v, int l) {
  return make_double2(read_lane(v.x, l), read_lane(v.y, l));
}
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
// Orders one wave's LDS accesses between phases that pass values across lanes.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Step 2. H (upper Hessenberg, from step 1) becomes the upper triangular Schur
// factor T, Z accumulates the rotations, w gets the eigenvalues t_jj.
//
// eig_schur_kernel (one workgroup per matrix) iterates on the active diagonal
// block [l, ihi] alone and records every sweep's rotations; eig_apply_kernel
// then applies the records to what the iteration never reads: Z, the rows
// above the active blocks and the columns right of them. The iteration is one
// dependent chain, so a matrix cannot fill more than a CU with it: with the
// whole of H and Z updated inside it (2 MB moved per sweep at n = 242, and two
// barriers per rotation), 96 matrices of order 242 took 142 ms. Only a sixth of
// that traffic belongs to the active blocks; the rest has no chain at all.
//
// A record: sweep q of a matrix is hdr[q] = {l, ihi, offset}, rotation k of it
// (rows and columns k, k + 1; l <= k < ihi) at offset + k - l of rotc / rots.
// A matrix whose record is full stops with its state saved (kState ints:
// ihi, its, done, info, sweeps, rotations) and goes on in the next launch.
//
// chase: one wave, rotations k0 .. k1 - 1 of a sweep on the block of rows and
// columns b0 .. b0 + bn - 1 (bn <= 64) in LDS, lane j on column j. A lane
// carries its column's value in the row that the next rotation takes, so a
// rotation is applied to all columns in two complex products; the three entries
// that decide the next rotation (rows k + 1, k + 2 of columns k, k + 1) are
// broadcast and turned at once by every lane. The column rotations of row r
// with index k >= r are left to apply_block_columns: no later rotation of the
// window reads them.
constexpr int kState = 8;
__device__ void chase(double2* __restrict__ blk, int ld, int bn, int b0, int k0, int k1, int l,
                      int ihi, double2 mu, double* __restrict__ rc, double2* __restrict__ rs) {
  const int lane = threadIdx.x & 63;
  int kk = k0 - b0;
  double2 x, y;
  if (k0 == l) {
    x = csub(blk[kk * ld + kk], mu);
    y = blk[kk * ld + kk + 1];
  } else {
    x = blk[(kk - 1) * ld + kk];
    y = blk[(kk - 1) * ld + kk + 1];
  }
  const bool live = lane < bn;
  double2* col = blk + min(lane, bn - 1) * ld;
  double2 cur = col[kk], nxt = col[kk + 1];
  double mc = 1.0;  // lane q keeps rotation k0 + q
  double2 ms = make_double2(0.0, 0.0);
  for (int k = k0; k < k1; ++k, ++kk) {
    double2 nn = col[min(kk + 2, bn - 1)];
    double c;
    double2 s, r;
    givens(x, y, c, s, r);
    const double2 cs = cconj(s);
    const bool keep = lane == k - k0;
    mc = keep ? c : mc;
    ms.x = keep ? s.x : ms.x;
    ms.y = keep ? s.y : ms.y;
    // row k, and r in the column before it (what the bulge leaves below the
    // subdiagonal is never read)
    double2 top = cadd(cscale(cur, c), cmul(s, nxt));
    const bool sub_col = lane == kk - 1;
    top.x = sub_col ? r.x : top.x;
    top.y = sub_col ? r.y : top.y;
    cur = csub(cscale(nxt, c), cmul(cs, cur));
    if (live && lane >= kk - 1 && (k > l || lane >= kk)) col[kk] = top;
    const double2 a = read_lane(cur, kk), b = read_lane(cur, kk + 1);
    double2 sub = read_lane(nn, kk + 1);
    if (k + 2 > ihi) sub = make_double2(0.0, 0.0);
    x = cadd(cscale(a, c), cmul(cs, b));
    y = cmul(cs, sub);
    const bool next = lane == kk + 1;
    const double2 nb = csub(cscale(b, c), cmul(s, a));
    cur.x = next ? nb.x : cur.x;
    cur.y = next ? nb.y : cur.y;
    nxt.x = next ? sub.x * c : nn.x;
    nxt.y = next ? sub.y * c : nn.y;
  }
  rc[lane] = mc;
  rs[lane] = ms;
  if (live && lane >= kk) col[kk] = cur;  // row k1
  if (lane == kk && k1 < ihi) col[kk + 1] = nxt;
  if (lane == 0) {
    blk[(kk - 1) * ld + kk] = x;
    if (k1 < ihi) blk[(kk - 1) * ld + kk + 1] = y;
  }
}

// The column rotations that chase left out: row b0 + row of the block takes
// rotations max(k0, b0 + row) .. k1 - 1.
__device__ inline void apply_block_columns(double2* __restrict__ blk, int ld, int row, int b0,
                                           int k0, int k1, const double* __restrict__ rc,
                                           const double2* __restrict__ rs) {
  constexpr int N = 4;  // rotations read ahead
  const int first = max(k0, b0 + row) - k0, nq = k1 - k0;
  double2* v = blk + (k0 - b0) * ld + row;  // v[q * ld]: column k0 + q
  double2 cur = v[0];
  for (int q0 = 0; q0 < nq; q0 += N) {
    double cx[N], cy[N], c[N], sx[N], sy[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {  // rotations nq and above are identities
      const int q = min(q0 + u, nq - 1);
      const double2 t = v[(q + 1) * ld], sv = rs[q0 + u];
      const bool on = q0 + u >= first;
      cx[u] = t.x;
      cy[u] = t.y;
      c[u] = on ? rc[q0 + u] : 1.0;
      sx[u] = on ? sv.x : 0.0;
      sy[u] = on ? sv.y : 0.0;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      if (q0 + u >= nq) break;
      const double2 o = make_double2(c[u] * cur.x + (sx[u] * cx[u] + sy[u] * cy[u]),
                                     c[u] * cur.y + (sx[u] * cy[u] - sy[u] * cx[u]));
      cur = make_double2(c[u] * cx[u] - (sx[u] * cur.x - sy[u] * cur.y),
                         c[u] * cy[u] - (sx[u] * cur.y + sy[u] * cur.x));
      v[(q0 + u) * ld] = o;
    }
  }
  v[nq * ld] = cur;
}

__device__ inline bool negligible(double sub, double tst, int n) {
  return sub <= fmax(DBL_MIN * ((double)n / DBL_EPSILON), DBL_EPSILON * tst);
}

// Wilkinson's shift of the trailing 2 x 2 block [[a, b], [c, d]]: its
// eigenvalue closer to d.
__device__ inline double2 wilkinson(double2 a, double2 b, double2 c, double2 d) {
  const double2 bc = cmul(b, c);
  const double2 x = cscale(csub(a, d), 0.5);
  double2 y = csqrt(cadd(cmul(x, x), bc));
  if (x.x * y.x + x.y * y.y < 0.0) y = make_double2(-y.x, -y.y);
  const double2 den = cadd(x, y);
  return (den.x == 0.0 && den.y == 0.0) ? d : csub(d, cdiv(bc, den));
}

// A window's W rotations (the last W - nq of them identities) on elements 0 .. nq
// of a row (COL) or a column, `stride` apart. Elements past nq are copies of
// the last; stored from the last down, its own value comes after theirs.
template <int W, bool COL>
__device__ inline void window_rotate(double2* __restrict__ v0, int stride, int nq,
                                     const double* rc, const double2* rs) {
  double vx[W + 1], vy[W + 1];
#pragma unroll
  for (int q = 0; q <= W; ++q) {
    const double2 t = v0[(size_t)(min(q, nq) * stride)];
    vx[q] = t.x;
    vy[q] = t.y;
  }
#pragma unroll
  for (int q = 0; q < W; ++q) {
    const double c = rc[q], sx = rs[q].x, sy = COL ? -rs[q].y : rs[q].y;
    const double ax = vx[q], ay = vy[q], bx = vx[q + 1], by = vy[q + 1];
    vx[q] = c * ax + (sx * bx - sy * by);
    vy[q] = c * ay + (sx * by + sy * bx);
    vx[q + 1] = c * bx - (sx * ax + sy * ay);
    vy[q + 1] = c * by - (sx * ay - sy * ax);
    // the rotations are read as they are used: all at once they would spill
    if (q % 4 == 3) asm volatile("" : "+v"(vx[q + 1]), "+v"(vy[q + 1]) : : "memory");
  }
  asm volatile("" : "+s"(nq));  // form the addresses again rather than keep them
#pragma unroll
  for (int q = W; q >= 0; --q) v0[(size_t)(min(q, nq) * stride)] = make_double2(vx[q], vy[q]);
}

// 96 matrices of order 242: 142 ms with everything in the iteration, now 42 ms
// for it and 11 ms for the three applications of its records.
//
// Two phases by the size of the active block. Above kInner it lives in memory
// and a sweep runs in windows of W rotations: the window's diagonal block (at
// most W + 3) is chased in LDS by one wave, then its rotations are applied in
// one pass to the active columns right of it and the active rows above it,
// one thread per column or row with the window's W + 1 values in registers.
// From kInner down the whole block stays in LDS and one wave runs every sweep.
template <int W, int kInner>
__global__ void __launch_bounds__(512)
eig_schur_kernel(int n, double2* __restrict__ Hall, double2* __restrict__ wall,
                 int* __restrict__ stateall, int capr, int caps, double* __restrict__ rotc,
                 double2* __restrict__ rots, int4* __restrict__ hdrall) {
  constexpr int LD = kInner + 1;
  static_assert(W + 3 <= kInner && kInner <= 64, "a block's columns are one wave's lanes");
  __shared__ double2 blk[LD * kInner];
  __shared__ double s_c[64];  // a lane each: identities past the last rotation
  __shared__ double2 s_s[64];
  __shared__ int s_l, s_ihi, s_its, s_stop, s_nsw, s_nrot;
  double2* H = Hall + blockIdx.x * (size_t)n * n;
  double2* w = wall + (size_t)blockIdx.x * n;
  int* state = stateall + (size_t)blockIdx.x * kState;
  rotc += (size_t)blockIdx.x * capr;
  rots += (size_t)blockIdx.x * capr;
  int4* hdr = hdrall + (size_t)blockIdx.x * caps;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (state[2]) {  // finished in an earlier launch
    if (tid == 0) state[4] = state[5] = 0;
    return;
  }
  int ihi = uniform(state[0]), its = uniform(state[1]), nsw = 0, nrot = 0, status = 0;
  bool full = false;
  while (ihi >= 0) {
    // largest k in [1, ihi] with a negligible subdiagonal: the active block is [l, ihi]
    if (tid == 0) s_l = 0;
    __syncthreads();
    for (int k = 1 + tid; k <= ihi; k += 512) {
      const double sub = cabs1(at(H, n, k, k - 1));
      double tst = cabs1(at(H, n, k - 1, k - 1)) + cabs1(at(H, n, k, k));
      if (tst == 0.0) {
        if (k >= 2) tst += fabs(at(H, n, k - 1, k - 2).x);
        if (k + 1 <= ihi) tst += fabs(at(H, n, k + 1, k).x);
      }
      if (negligible(sub, tst, n)) atomicMax(&s_l, k);
    }
    __syncthreads();
    const int l = uniform(s_l);
    __syncthreads();  // every thread has read s_l before it is reset
    if (l > 0 && tid == 0) at(H, n, l, l - 1) = make_double2(0.0, 0.0);
    if (l == ihi) {  // a 1 x 1 block: eigenvalue ihi has converged
      if (tid == 0) w[ihi] = at(H, n, ihi, ihi);
      --ihi;
      its = 0;
      __syncthreads();
      continue;
    }
    const int m = ihi - l + 1;
    if (m <= kInner) {
      for (int e = tid; e < m * m; e += 512) {
        const int r = e % m, c = e / m;
        blk[c * LD + r] = at(H, n, l + r, l + c);
      }
      __syncthreads();
      if (wave == 0) {
        int hi = ihi, stop = 0;
        while (hi >= l) {
          wave_sync();
          // lane q tests the subdiagonal of row l + q
          bool neg = false;
          const int q = lane, top = hi - l;
          if (q >= 1 && q <= top) {
            const double sub = cabs1(blk[(q - 1) * LD + q]);
            double tst = cabs1(blk[(q - 1) * LD + q - 1]) + cabs1(blk[q * LD + q]);
            if (tst == 0.0) {
              if (q >= 2) tst += fabs(blk[(q - 2) * LD + q - 1].x);
              if (q + 1 <= top) tst += fabs(blk[q * LD + q + 1].x);
            }
            neg = negligible(sub, tst, n);
          }
          const unsigned long long mask = __ballot(neg);
          const int dl = uniform(mask ? 63 - __clzll((long long)mask) : 0);
          const int al = l + dl;  // the active block is [al, hi]
          if (dl > 0 && lane == 0) blk[(dl - 1) * LD + dl] = make_double2(0.0, 0.0);
          if (al == hi) {
            if (lane == 0) w[hi] = blk[dl * LD + dl];
            --hi;
            its = 0;
            continue;
          }
          if (nrot + (hi - al) > capr || nsw >= caps) {
            stop = 1;
            break;
          }
          if (++its > kMaxSweepsPerEigenvalue) {
            stop = 2;
            break;
          }
          double2* sb = blk + dl * (LD + 1);
          const int bn = hi - al + 1;
          double2 mu;
          if (its % 20 == 10) {
            mu = cadd(sb[0], make_double2(0.75 * fabs(sb[1].x), 0.0));
          } else if (its % 20 == 0) {
            mu = cadd(sb[(bn - 1) * (LD + 1)],
                      make_double2(0.75 * fabs(sb[(bn - 2) * LD + bn - 1].x), 0.0));
          } else {
            mu = wilkinson(sb[(bn - 2) * (LD + 1)], sb[(bn - 1) * LD + bn - 2],
                           sb[(bn - 2) * LD + bn - 1], sb[(bn - 1) * (LD + 1)]);
          }
          chase(sb, LD, bn, al, al, hi, al, hi, mu, s_c, s_s);
          wave_sync();
          if (lane < bn) apply_block_columns(sb, LD, lane, al, al, hi, s_c, s_s);
          wave_sync();
          if (lane < bn - 1) {
            rotc[nrot + lane] = s_c[lane];
            rots[nrot + lane] = s_s[lane];
          }
          if (lane == 0) hdr[nsw] = make_int4(al, hi, nrot, 0);
          nrot += hi - al;
          ++nsw;
        }
        if (lane == 0) {
          s_ihi = hi;
          s_its = its;
          s_stop = stop;
          s_nsw = nsw;
          s_nrot = nrot;
        }
      }
      __syncthreads();
      for (int e = tid; e < m * m; e += 512) {
        const int r = e % m, c = e / m;
        at(H, n, l + r, l + c) = blk[c * LD + r];
      }
      ihi = uniform(s_ihi);
      its = uniform(s_its);
      nsw = uniform(s_nsw);
      nrot = uniform(s_nrot);
      const int stop = uniform(s_stop);
      __syncthreads();
      if (stop == 2) status = ihi + 1;
      full = stop == 1;
      if (stop) break;
      continue;
    }
    if (nrot + (ihi - l) > capr || nsw >= caps) {
      full = true;
      break;
    }
    if (++its > kMaxSweepsPerEigenvalue) {
      status = ihi + 1;
      break;
    }
    double2 mu;
    if (its % 20 == 10)
      mu = cadd(at(H, n, l, l), make_double2(0.75 * fabs(at(H, n, l + 1, l).x), 0.0));
    else if (its % 20 == 0)
      mu = cadd(at(H, n, ihi, ihi), make_double2(0.75 * fabs(at(H, n, ihi, ihi - 1).x), 0.0));
    else
      mu = wilkinson(at(H, n, ihi - 1, ihi - 1), at(H, n, ihi - 1, ihi), at(H, n, ihi, ihi - 1),
                     at(H, n, ihi, ihi));
    // one implicit single-shift QR sweep over [l, ihi], W rotations per window
    for (int k0 = l; k0 < ihi; k0 += W) {
      const int k1 = min(k0 + W, ihi);      // rotations k0 .. k1 - 1
      const int b0 = k0 == l ? l : k0 - 1;  // block rows and columns b0 .. be
      const int be = min(k1 + 1, ihi);
      const int bn = be - b0 + 1, nq = k1 - k0;
      for (int e = tid; e < bn * bn; e += 512) {
        const int r = e % bn, c = e / bn;
        blk[c * LD + r] = at(H, n, b0 + r, b0 + c);
      }
      __syncthreads();
      if (wave == 0) chase(blk, LD, bn, b0, k0, k1, l, ihi, mu, s_c, s_s);
      __syncthreads();
      if (wave == 0) {  // the block itself, and the record
        if (lane < bn) {
          apply_block_columns(blk, LD, lane, b0, k0, k1, s_c, s_s);
          for (int c = 0; c < bn; ++c) at(H, n, b0 + lane, b0 + c) = blk[c * LD + lane];
        }
        if (lane < nq) {
          rotc[nrot + (k0 - l) + lane] = s_c[lane];
          rots[nrot + (k0 - l) + lane] = s_s[lane];
        }
      } else {
        // columns right of the block, then rows above it
        const int nright = ihi - be, nabove = b0 - l;
        for (int i = tid - 64; i < nright; i += 448)
          window_rotate<W, false>(&at(H, n, k0, be + 1 + i), 1, nq, s_c, s_s);
        for (int i = 511 - tid; i < nabove; i += 448)
          window_rotate<W, true>(&at(H, n, l + i, k0), n, nq, s_c, s_s);
      }
      __syncthreads();
    }
    if (tid == 0) hdr[nsw] = make_int4(l, ihi, nrot, 0);
    nrot += ihi - l;
    ++nsw;
  }
  if (tid == 0) {
    state[0] = ihi;
    state[1] = its;
    state[2] = full ? 0 : 1;
    state[3] = status;
    state[4] = nsw;
    state[5] = nrot;
  }
}

__global__ void eig_schur_begin(int n, int count, int* __restrict__ state) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= count) return;
  int* s = state + (size_t)b * kState;
  s[0] = n - 1;
  for (int i = 1; i < kState; ++i) s[i] = 0;
}

// The recorded sweeps on what the iteration left out. MODE 0: every row of Z
// (column rotations). MODE 1: row r of H takes the sweeps with l > r (column
// rotations). MODE 2: column j of H takes the sweeps with ihi < j (row
// rotations). A row of H right of one block and above another takes both; they
// act from different sides and commute.
//
// One wave per 64 rows (columns), a lane each. Sixteen sweeps run at once in a
// skewed order: at step t sweep s applies its rotation k = t - s to the elements
// k and k + 1. Of its two results the one at k is the second element of sweep
// s + 1, next in the same step, the one at k + 1 its own first element at the
// next step; so the sixteen form a pipeline held in registers, into which one
// element enters per step and from which one leaves. An element is read and written once per sixteen
// sweeps. A rotation outside its sweep's range is an identity. The next
// chunk's elements and rotations are fetched during a chunk of 16 steps.
// Bound by the FP64 units: 12 operations per rotation and lane. (With the
// elements in an LDS ring, each rotation reading and writing two: 23.5 ms
// instead of 10.9 for the three kernels on 96 matrices of order 242.)
constexpr int kApplySweeps = 16, kApplySteps = 16;
template <int MODE>
__global__ void __launch_bounds__(64)
eig_apply_kernel(int n, double2* __restrict__ Mall, const int* __restrict__ stateall, int capr,
                 int caps, const double* __restrict__ rotc, const double2* __restrict__ rots,
                 const int4* __restrict__ hdrall) {
  constexpr int S = kApplySweeps, T = kApplySteps;
  static_assert(T == 16 && S == 16, "fetch layout");
  __shared__ double2 s_in[T][64];
  __shared__ double s_c[T * S];
  __shared__ double2 s_s[T * S];
  const int lane = threadIdx.x, b = blockIdx.y;
  const int first = blockIdx.x * 64, id = first + lane, last = min(first + 63, n - 1);
  double2* M = Mall + (size_t)b * n * n;
  rotc += (size_t)b * capr;
  rots += (size_t)b * capr;
  const int4* hdr = hdrall + (size_t)b * caps;
  const int nsw = uniform(stateall[(size_t)b * kState + 4]);
  // element q of this lane's row or column
  const size_t stride = MODE == 2 ? 1 : (size_t)n;
  double2* base = M + (MODE == 2 ? (size_t)min(id, n - 1) * n : (size_t)min(id, n - 1));
  for (int s0 = 0; s0 < nsw; s0 += S) {
    // lane u of each 16 holds sweep s0 + u (an empty range past the last)
    const int4 h = hdr[min(s0 + (lane & 15), nsw - 1)];
    int el = h.x, eh = h.y;
    const bool on = s0 + (lane & 15) < nsw && (MODE == 0 || (MODE == 1 ? first < el : last > eh));
    if (!__ballot(on)) continue;
    if (!on) eh = el;
    // the group's range, and this lane's sweeps (bit s: it takes part in sweep s)
    int lo = on ? el : n, hi = on ? eh : 0;
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) {
      lo = min(lo, __shfl_xor(lo, o, 64));
      hi = max(hi, __shfl_xor(hi, o, 64));
    }
    lo = uniform(lo);
    hi = uniform(hi);
    unsigned takes = 0xffffu;
    if (MODE != 0) {
      takes = 0;
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (MODE == 1 ? id < __shfl(h.x, s, 64) : id > __shfl(h.y, s, 64)) takes |= 1u << s;
    }
    double colx[T], coly[T], rcv[4], rsx[4], rsy[4];
    double px[S], py[S];  // sweep s's first element at step t: t - s
#pragma unroll
    for (int s = 0; s < S; ++s) px[s] = py[s] = 0.0;
    {
      const double2 v = base[(size_t)lo * stride];
      px[0] = v.x;
      py[0] = v.y;
    }
    // the pass before the first only loads
    for (int t0 = lo - T; t0 - S + 1 <= hi; t0 += T) {
      const bool run = t0 >= lo;
      if (run) {
#pragma unroll
        for (int i = 0; i < T; ++i) s_in[i][lane] = make_double2(colx[i], coly[i]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          s_c[q * 64 + lane] = rcv[q];
          s_s[q * 64 + lane] = make_double2(rsx[q], rsy[q]);
        }
      }
      wave_sync();
      // elements t + 1 of the next chunk's steps, and its rotations: step
      // 4 q + lane / 16 of sweep lane % 16 at q * 64 + lane
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const double2 v = base[(size_t)min(t0 + T + 1 + i, hi) * stride];
        colx[i] = v.x;
        coly[i] = v.y;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = t0 + T + 4 * q + (lane >> 4) - (lane & 15);
        const bool in = k >= el && k < eh;
        const int e = in ? h.z + k - el : 0;
        const double2 v = rots[e];
        const double c = rotc[e];
        rcv[q] = in ? c : 1.0;
        rsx[q] = in ? v.x : 0.0;
        rsy[q] = in ? (MODE == 2 ? v.y : -v.y) : 0.0;
      }
      if (!run) continue;
#pragma unroll 1
      for (int i = 0; i < T; ++i) {
        const double2 in = s_in[i][lane];
        double fx = in.x, fy = in.y;  // the element handed down: sweep s's second
#pragma unroll
        for (int s = 0; s < S; ++s) {
          double c = s_c[i * S + s];
          const double2 sv = s_s[i * S + s];
          double sx = sv.x, sy = sv.y;
          if (MODE != 0) {
            const bool mine = (takes >> s) & 1;
            c = mine ? c : 1.0;
            sx = mine ? sx : 0.0;
            sy = mine ? sy : 0.0;
          }
          const double ax = px[s], ay = py[s];
          // first: c a + s f; second: c f - conj(s) a
          const double ox = c * ax + (sx * fx - sy * fy), oy = c * ay + (sx * fy + sy * fx);
          px[s] = c * fx - (sx * ax + sy * ay);
          py[s] = c * fy - (sx * ay - sy * ax);
          fx = ox;
          fy = oy;
        }
        const int q = t0 + i - S + 1;  // the element that leaves the last sweep
        if (q >= lo && q <= hi && id < n) base[(size_t)q * stride] = make_double2(fx, fy);
      }
      wave_sync();
    }
  }
}

// Column-major T -> row-major copy of its upper triangle (zeros below), in
// 32 x 32 tiles through LDS.
__global__ void __launch_bounds__(256)
eig_transpose_kernel(int n, const double2* __restrict__ T, double2* __restrict__ Tt) {
  __shared__ double2 tile[32][33];
  const size_t nn = (size_t)n * n;
  const double2* src = T + blockIdx.z * nn;
  double2* dst = Tt + blockIdx.z * nn;
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int j = ty; j < 32; j += 8) {
    const int r = r0 + tx, c = c0 + j;
    tile[j][tx] = (r < n && c < n && r <= c) ? src[(size_t)c * n + r] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  for (int j = ty; j < 32; j += 8) {
    const int r = r0 + j, c = c0 + tx;
    if (r < n && c < n) dst[(size_t)r * n + c] = tile[tx][j];
  }
}

// Step 3. One wavefront per eigenvector j of one matrix: lane l holds
// y(64 t + l) in slot t (n <= 64 NS). Row i of T (row-major Tt) against y,
// summed over the wave, gives y(i) = -(sum_{k>i} t_ik y(k)) / (t_ii - t_jj)
// for i = j-1 .. 0; the result goes to column j of Y (zeros below j).
template <int NS>
__global__ void __launch_bounds__(256)
eig_vectors_kernel(int n, int count, const double2* __restrict__ Tt,
                   const double2* __restrict__ wall, double2* __restrict__ Y) {
  const int lane = threadIdx.x & 63;
  const long long gw = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (gw >= (long long)count * n) return;
  const int b = (int)(gw / n), j = (int)(gw % n);
  const size_t nn = (size_t)n * n;
  const double2* T = Tt + b * nn;
  const double2 lam = wall[(size_t)b * n + j];
  const double smin = fmax(DBL_EPSILON * cabs1(lam), DBL_MIN * ((double)n / DBL_EPSILON));
  double2 y[NS];
#pragma unroll
  for (int t = 0; t < NS; ++t) y[t] = make_double2(64 * t + lane == j ? 1.0 : 0.0, 0.0);
  for (int i = j - 1; i >= 0; --i) {
    const double2* row = T + (size_t)i * n;
    double2 acc = make_double2(0.0, 0.0);
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int k = 64 * t + lane;
      if (k > i && k <= j) acc = cadd(acc, cmul(row[k], y[t]));
    }
    acc = wave_sum(acc);
    double2 d = csub(row[i], lam);
    if (cabs1(d) < smin) d = make_double2(smin, 0.0);
    const double2 yi = cdiv(make_double2(-acc.x, -acc.y), d);
#pragma unroll
    for (int t = 0; t < NS; ++t)
      if (64 * t + lane == i) y[t] = yi;
  }
  double2* out = Y + b * nn + (size_t)j * n;
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    const int k = 64 * t + lane;
    if (k < n) out[k] = k <= j ? y[t] : make_double2(0.0, 0.0);
  }
}

// Unit 2-norm columns, one wavefront per column.
__global__ void __launch_bounds__(256)
eig_normalize_kernel(int n, long long ncols, double2* __restrict__ X) {
  const int lane = threadIdx.x & 63;
  const long long col = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= ncols) return;
  double2* x = X + col * n;
  double s = 0.0;
  for (int i = lane; i < n; i += 64) s += x[i].x * x[i].x + x[i].y * x[i].y;
  for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
  const double inv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
  for (int i = lane; i < n; i += 64) x[i] = cscale(x[i], inv);
}

// Columns scaled by one complex factor each: X[:, j] *= f[j], [count][n] factors.
__global__ void __launch_bounds__(256)
eig_scale_cols_kernel(int n, long long ncols, const double2* __restrict__ f,
                      double2* __restrict__ X) {
  const int lane = threadIdx.x & 63;
  const long long col = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= ncols) return;
  const double2 g = f[col];
  double2* x = X + col * n;
  for (int i = lane; i < n; i += 64) x[i] = cmul(x[i], g);
}

}  // namespace

size_t eig_hessenberg_work(int n) { return hess_work(n) * sizeof(double2); }

hipError_t launch_eig_hessenberg(int n, int count, double* A, double* Z, double* work,
                                 hipStream_t s) {
  if (n < 1 || n > kEigMaxN || count < 1) return hipErrorInvalidValue;
  const size_t lds = ((size_t)n + 1024) * sizeof(double2);
  double2* a = reinterpret_cast<double2*>(A);
  double2* z = reinterpret_cast<double2*>(Z);
  double2* w = reinterpret_cast<double2*>(work);
  if (n > 2) eig_hessenberg_kernel<<<count, 1024, lds, s>>>(n, a, w);
  eig_hess_apply_kernel<<<dim3((n + 63) / 64, count, 2), 256, 0, s>>>(n, a, z, w);
  if (n > 2) eig_hess_clear_kernel<<<dim3(n, count), 256, 0, s>>>(n, a);
  return hipGetLastError();
}

hipError_t launch_eig_schur_begin(int n, int count, int* state, hipStream_t s) {
  if (n < 1 || n > kEigMaxN || count < 1) return hipErrorInvalidValue;
  eig_schur_begin<<<(count + 63) / 64, 64, 0, s>>>(n, count, state);
  return hipGetLastError();
}

hipError_t launch_eig_schur(int n, int count, double* H, double* Z, double* w,
                            const EigRecord& rec, hipStream_t s) {
  if (n < 1 || n > kEigMaxN || count < 1) return hipErrorInvalidValue;
  double2* h = reinterpret_cast<double2*>(H);
  double2* z = reinterpret_cast<double2*>(Z);
  double2* rs = reinterpret_cast<double2*>(rec.rots);
  int4* hdr = reinterpret_cast<int4*>(rec.hdr);
  eig_schur_kernel<kEigWindow, kEigInner><<<count, 512, 0, s>>>(
      n, h, reinterpret_cast<double2*>(w), rec.state, rec.capr, rec.caps, rec.rotc, rs, hdr);
  const dim3 grid((n + 63) / 64, count);
  eig_apply_kernel<0><<<grid, 64, 0, s>>>(n, z, rec.state, rec.capr, rec.caps, rec.rotc, rs, hdr);
  eig_apply_kernel<1><<<grid, 64, 0, s>>>(n, h, rec.state, rec.capr, rec.caps, rec.rotc, rs, hdr);
  eig_apply_kernel<2><<<grid, 64, 0, s>>>(n, h, rec.state, rec.capr, rec.caps, rec.rotc, rs, hdr);
  return hipGetLastError();
}

hipError_t launch_eig_vectors(int n, int count, const double* T, double* Tt, const double* w,
                              double* Y, hipStream_t s) {
  if (n < 1 || n > kEigMaxN || count < 1) return hipErrorInvalidValue;
  const unsigned tiles = (unsigned)((n + 31) / 32);
  eig_transpose_kernel<<<dim3(tiles, tiles, count), 256, 0, s>>>(
      n, reinterpret_cast<const double2*>(T), reinterpret_cast<double2*>(Tt));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const long long waves = (long long)count * n;
  const unsigned blocks = (unsigned)((waves + 3) / 4);
  const double2* tt = reinterpret_cast<const double2*>(Tt);
  const double2* ww = reinterpret_cast<const double2*>(w);
  double2* y = reinterpret_cast<double2*>(Y);
  const int ns = (n + 63) / 64;
  if (ns <= 2) eig_vectors_kernel<2><<<blocks, 256, 0, s>>>(n, count, tt, ww, y);
  else if (ns <= 4) eig_vectors_kernel<4><<<blocks, 256, 0, s>>>(n, count, tt, ww, y);
  else if (ns <= 8) eig_vectors_kernel<8><<<blocks, 256, 0, s>>>(n, count, tt, ww, y);
  else if (ns <= 16) eig_vectors_kernel<16><<<blocks, 256, 0, s>>>(n, count, tt, ww, y);
  else eig_vectors_kernel<32><<<blocks, 256, 0, s>>>(n, count, tt, ww, y);
  return hipGetLastError();
}

hipError_t launch_eig_normalize(int n, long long ncols, double* X, hipStream_t s) {
  if (ncols <= 0) return hipSuccess;
  eig_normalize_kernel<<<(unsigned)((ncols + 3) / 4), 256, 0, s>>>(
      n, ncols, reinterpret_cast<double2*>(X));
  return hipGetLastError();
}

hipError_t launch_eig_scale_cols(int n, long long ncols, const double* f, double* X,
                                 hipStream_t s) {
  if (ncols <= 0) return hipSuccess;
  eig_scale_cols_kernel<<<(unsigned)((ncols + 3) / 4), 256, 0, s>>>(
      n, ncols, reinterpret_cast<const double2*>(f), reinterpret_cast<double2*>(X));
  return hipGetLastError();
}

}  // namespace scw
