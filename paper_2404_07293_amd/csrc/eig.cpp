// Host driver of the batched device eigensolver (kernels_eig.hip) and its C
// ABI entry point scw_eig_batched: Hessenberg reduction, Schur form and the
// Schur factor's eigenvectors per matrix, then X = Z Y for the whole batch as
// one strided-batched complex GEMM and unit-norm columns.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <algorithm>
#include <string>
#include <vector>

#include "scw_internal.h"

namespace scw {

int blas_fail(const char* call, int status) {
  const rocblas_status st = static_cast<rocblas_status>(status);
  const bool memory = st == rocblas_status_memory_error;
  if (memory) (void)hipGetLastError();
  return fail(memory ? SCW_ENOMEM : SCW_EHIP,
              std::string(call) + ": " + rocblas_status_to_string(st));
}

int blas_handle(Context& ctx, hipStream_t st, void** out) {
  if (!ctx.blas) {
    rocblas_handle h = nullptr;
    const rocblas_status r = rocblas_create_handle(&h);
    if (r != rocblas_status_success) return blas_fail("rocblas_create_handle", r);
    ctx.blas = h;
  }
  rocblas_handle h = static_cast<rocblas_handle>(ctx.blas);
  const rocblas_status r = rocblas_set_stream(h, st);
  if (r != rocblas_status_success) return blas_fail("rocblas_set_stream", r);
  *out = h;
  return SCW_OK;
}

namespace {
// The eigensolver's workspace, one allocation (each costs microseconds) of six
// regions, each for all matrices: Z, the row-major copy, the states, the sweep
// headers, the reduction's panels where they need more than the row-major copy's
// region (free until the iteration is done), and the rotations. Matrices that
// stay in LDS get room for the rotations of a whole iteration, as another launch
// costs more than their sweeps (100 matrices of order 8: 370 us a call, 562 in
// four launches; 16 of order 50: 3.86 ms, 4.23).
struct EigWork {
  size_t part[6];  // bytes per matrix
  size_t capr;
  int caps;
  explicit EigWork(int n) {
    const size_t nn = (size_t)n * n;
    capr = n <= 64 ? 2 * nn + 64 : nn / 2 + n;
    caps = 4 * n + 64;
    const size_t hess = eig_hessenberg_work(n);
    const size_t p[6] = {nn * 16, nn * 16, 8 * sizeof(int), (size_t)caps * 16,
                         hess > nn * 16 ? hess : 0, capr * 24};
    std::copy(p, p + 6, part);
  }
  size_t at(size_t count, int k) const {  // offset of region k, 256-byte aligned
    size_t o = 0;
    for (int i = 0; i < k; ++i) o += (part[i] * count + 255) / 256 * 256;
    return o;
  }
};
}  // namespace

size_t eig_matrix_bytes(int n) {
  const EigWork wk(n);
  return wk.at(1, 6);
}

int device_eig_batched(Context& ctx, int n, int count, double* A, double* w, double* X,
                       hipStream_t st) {
  if (n < 1 || n > kEigMaxN || count < 1)
    return fail(SCW_EINVAL, "batched eigensolver: n must be in 1.." + std::to_string(kEigMaxN) +
                                " and count positive");
  if (!A || !w || !X) return fail(SCW_EINVAL, "batched eigensolver: null pointer");
  SCW_HIP(hipSetDevice(ctx.device));
  const size_t nn = (size_t)n * n;
  const EigWork wk(n);
  // A usual iteration has about 1.25 n^2 rotations per matrix and takes three
  // launches with a record of n^2 / 2; another launch costs tens of microseconds,
  // so less is taken where memory is short.
  EigRecord rec{};
  size_t capr = wk.capr;
  rec.caps = wk.caps;
  const size_t o_tt = wk.at(count, 1), o_state = wk.at(count, 2), o_hdr = wk.at(count, 3),
               o_hess = wk.part[4] ? wk.at(count, 4) : o_tt, o_rot = wk.at(count, 5);
  DevBuf work;
  int rc;
  while ((rc = work.reserve(o_rot + capr * 24 * count)) == SCW_ENOMEM && capr > (size_t)n)
    capr = std::max<size_t>(n, capr / 4);
  if (rc) return rc;
  char* base = work.as<char>();
  double* Z = reinterpret_cast<double*>(base);
  double* Tt = reinterpret_cast<double*>(base + o_tt);
  double* hwork = reinterpret_cast<double*>(base + o_hess);
  rec.capr = (int)capr;
  rec.state = reinterpret_cast<int*>(base + o_state);
  rec.hdr = reinterpret_cast<int*>(base + o_hdr);
  rec.rots = reinterpret_cast<double*>(base + o_rot);
  rec.rotc = rec.rots + 2 * capr * count;
  SCW_HIP(launch_eig_hessenberg(n, count, A, Z, hwork, st));
  SCW_HIP(launch_eig_schur_begin(n, count, rec.state, st));
  std::vector<int> state(8 * (size_t)count);
  for (bool done = false; !done;) {
    SCW_HIP(launch_eig_schur(n, count, A, Z, w, rec, st));
    SCW_HIP(hipMemcpyAsync(state.data(), rec.state, state.size() * sizeof(int),
                           hipMemcpyDeviceToHost, st));
    SCW_HIP(hipStreamSynchronize(st));
    done = true;
    for (int b = 0; b < count; ++b) done = done && state[8 * (size_t)b + 2] != 0;
  }
  for (int b = 0; b < count; ++b)
    if (state[8 * (size_t)b + 3])
      return fail(SCW_ELAPACK, "batched eigensolver: QR iteration of matrix " +
                                   std::to_string(b) + " did not converge at eigenvalue " +
                                   std::to_string(state[8 * (size_t)b + 3] - 1));
  // the Schur factor's eigenvectors overwrite A once it is copied row-major
  SCW_HIP(launch_eig_vectors(n, count, A, Tt, w, A, st));
  void* hv = nullptr;
  if ((rc = blas_handle(ctx, st, &hv))) return rc;
  rocblas_handle h = static_cast<rocblas_handle>(hv);
  const rocblas_double_complex one = {1.0, 0.0}, zero = {0.0, 0.0};
  const rocblas_status bs = rocblas_zgemm_strided_batched(
      h, rocblas_operation_none, rocblas_operation_none, n, n, n, &one,
      reinterpret_cast<const rocblas_double_complex*>(Z), n, (rocblas_stride)nn,
      reinterpret_cast<const rocblas_double_complex*>(A), n, (rocblas_stride)nn, &zero,
      reinterpret_cast<rocblas_double_complex*>(X), n, (rocblas_stride)nn, count);
  if (bs != rocblas_status_success) return blas_fail("rocblas_zgemm_strided_batched", bs);
  SCW_HIP(launch_eig_normalize(n, (long long)count * n, X, st));
  SCW_HIP(hipStreamSynchronize(st));
  return SCW_OK;
}

}  // namespace scw

using namespace scw;

extern "C" int scw_eig_batched(scw_ctx* ctx, int n, int count, double* A_dev, double* w_dev,
                               double* X_dev, void* hip_stream) {
  if (!ctx) return fail(SCW_EINVAL, "null context");
  return device_eig_batched(ctx->c, n, count, A_dev, w_dev, X_dev,
                            reinterpret_cast<hipStream_t>(hip_stream));
}
