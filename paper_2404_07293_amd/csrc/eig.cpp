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

int device_eig_batched(Context& ctx, int n, int count, double* A, double* w, double* X,
                       hipStream_t st) {
  if (n < 1 || n > kEigMaxN || count < 1)
    return fail(SCW_EINVAL, "batched eigensolver: n must be in 1.." + std::to_string(kEigMaxN) +
                                " and count positive");
  if (!A || !w || !X) return fail(SCW_EINVAL, "batched eigensolver: null pointer");
  SCW_HIP(hipSetDevice(ctx.device));
  const size_t nn = (size_t)n * n;
  DevBuf dZ, dTt, dstate, drot, dhdr;
  int rc;
  // A usual iteration has about 1.25 n^2 rotations per matrix and takes three
  // launches with this record; another launch costs tens of microseconds, so
  // less is taken where memory is short.
  EigRecord rec{};
  size_t capr = nn / 2 + n;
  rec.caps = 4 * n + 64;
  if ((rc = dZ.reserve(nn * 16 * count)) || (rc = dTt.reserve(nn * 16 * count)) ||
      (rc = dstate.reserve(sizeof(int) * 8 * count)) ||
      (rc = dhdr.reserve((size_t)rec.caps * 16 * count)))
    return rc;
  while ((rc = drot.reserve(capr * 24 * count)) == SCW_ENOMEM && capr > (size_t)n)
    capr = std::max<size_t>(n, capr / 4);
  if (rc) return rc;
  rec.capr = (int)capr;
  rec.state = dstate.as<int>();
  rec.rots = drot.as<double>();
  rec.rotc = drot.as<double>() + 2 * capr * count;
  rec.hdr = dhdr.as<int>();
  // the row-major copy's buffer is free until the iteration is done; small
  // matrices need more for the reduction's panels than it holds
  DevBuf dhess;
  double* hwork = dTt.as<double>();
  if (eig_hessenberg_work(n) > nn * 16) {
    if ((rc = dhess.reserve(eig_hessenberg_work(n) * count))) return rc;
    hwork = dhess.as<double>();
  }
  SCW_HIP(launch_eig_hessenberg(n, count, A, dZ.as<double>(), hwork, st));
  SCW_HIP(launch_eig_schur_begin(n, count, rec.state, st));
  std::vector<int> state(8 * (size_t)count);
  for (bool done = false; !done;) {
    SCW_HIP(launch_eig_schur(n, count, A, dZ.as<double>(), w, rec, st));
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
  SCW_HIP(launch_eig_vectors(n, count, A, dTt.as<double>(), w, A, st));
  void* hv = nullptr;
  if ((rc = blas_handle(ctx, st, &hv))) return rc;
  rocblas_handle h = static_cast<rocblas_handle>(hv);
  const rocblas_double_complex one = {1.0, 0.0}, zero = {0.0, 0.0};
  const rocblas_status bs = rocblas_zgemm_strided_batched(
      h, rocblas_operation_none, rocblas_operation_none, n, n, n, &one,
      reinterpret_cast<const rocblas_double_complex*>(dZ.p), n, (rocblas_stride)nn,
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
