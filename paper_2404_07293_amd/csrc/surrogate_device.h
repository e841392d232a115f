// Device helpers shared by the surrogate's kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace scw {
namespace {

struct f2 {
  float x, y;
};

typedef float floatx16 __attribute__((ext_vector_type(16)));

// a patch's side, the layers' spectral half plane and the channel count
constexpr int SN = 32, SKY = 17, SKX = 9, SNM = SKY * SKX, SW = 32;

// Loads and stores, non-temporal with NT.
template <bool NT, typename V>
__device__ __forceinline__ V ld(const V* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, typename V>
__device__ __forceinline__ void st(V* p, V v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// Orders one wave's LDS accesses between phases that pass values across lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// round to bf16, nearest even, by the hardware's conversion (two values per
// instruction where the compiler pairs them)
__device__ __forceinline__ float rbf(float x) { return (float)(__bf16)x; }
template <bool BF16>
__device__ __forceinline__ float op(float x) { return BF16 ? rbf(x) : x; }
template <bool BF16>
__device__ __forceinline__ f2 op(f2 x) { return BF16 ? f2{rbf(x.x), rbf(x.y)} : x; }

// d GELU / dz for the backward pass (exact erf)
__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.f + erff(z * 0.70710678118654752f)) +
         z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

}  // namespace
}  // namespace scw
