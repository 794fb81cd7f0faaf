// FP64 multiply-add and Horner forms with scalar-register coefficients, shared
// by the device code of wl_kernels.hip and wl_generate.hip.
#pragma once

#include <hip/hip_runtime.h>

namespace wl {

// acc * v + c as the three-address v_fma_f64 with the coefficient c in a
// scalar register pair.  Polynomial coefficients as vector operands are
// loop-invariant values the compiler holds in vector registers across the
// segment walk (two per coefficient: 53 in the FP64 walk's polynomials, 16
// more in the per-loop cosine), which under a register budget are spilled to
// scratch and reloaded for every loop or segment; as scalar operands they
// sit in scalar registers (constant-memory loads, or two s_mov each) and the
// FMA reads them directly.  (The two-address v_fmac_f64 would overwrite its
// addend, so a coefficient addend would first be copied into a vector
// register at every step.)
__device__ __forceinline__ double fma3s_f64(double acc, double v, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(acc), "v"(v), "s"(c));
  return r;
}

// Horner with every coefficient in scalar registers, for the per-loop
// epilogue (between segment walks, where any vector register held across
// the walk is spilled).  The first step is c[DEG] v (rounded) + c[DEG-1]:
// an FMA of two constants would need two scalar operands, which a VOP3
// instruction on this chip cannot read.
template <int DEG>
__device__ __forceinline__ double horner_s_f64(const double (&c)[DEG + 1], double v) {
  double t, acc;
  asm("v_mul_f64 %0, %1, %2" : "=v"(t) : "v"(v), "s"(c[DEG]));
  asm("v_add_f64 %0, %1, %2" : "=v"(acc) : "v"(t), "s"(c[DEG - 1]));
#pragma unroll
  for (int k = DEG - 2; k >= 0; --k) acc = fma3s_f64(acc, v, c[k]);
  return acc;
}

}  // namespace wl
