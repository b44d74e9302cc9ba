// Device helpers shared by the solver kernels: epoch-tagged exchange words,
// cross-lane sums and the IRLS weights.
#pragma once

#include "kf_internal.h"

namespace kf {

__device__ inline void st_word(KF_GLOBAL uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint64_t ld_word(const KF_GLOBAL uint64_t* p) {
  return __hip_atomic_load(const_cast<KF_GLOBAL uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Compiler-only barrier (no instruction): the value counts as redefined here,
// so per-pixel addresses derived from it are recomputed inside the loop that
// holds the barrier instead of being hoisted and kept live in registers for the
// whole launch (that cut the register count per pixel from ~53 to ~16).
__device__ inline void refresh(int& v) { asm volatile("" : "+v"(v)); }

__device__ inline uint64_t tagged(uint32_t bits, uint32_t e) { return ((uint64_t)e << 32) | (uint64_t)bits; }

// One-word transport of an FP64 partial: the top 48 bits of the double
// (rounded; relative precision 2^-37) and a 16-bit epoch. Used when a launch
// spans fewer than 30000 epochs, so a slot's previous content is never 2^16
// epochs old.
struct Packed48 {
  __device__ static uint64_t make_word(double v, uint32_t e) {
    const uint64_t b = (uint64_t)__double_as_longlong(v) + 0x8000ull;
    return ((uint64_t)(e & 0xffffu) << 48) | (b >> 16);
  }
  __device__ static bool ready(uint64_t w, uint32_t e) { return (uint32_t)(w >> 48) == (e & 0xffffu); }
  __device__ static double value(uint64_t w) {
    return __longlong_as_double((long long)((w & 0xffffffffffffull) << 16));
  }
};

// v as it is, not to be fused with what uses it.
template <typename T>
__device__ inline T rounded(T v) {
  asm("" : "+v"(v));
  return v;
}

// Data-parallel-primitive move of both halves of a double (out-of-row lanes read 0).
template <int CTRL, int ROW_MASK, bool BOUND_ZERO>
__device__ inline double dpp_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROW_MASK, 0xf, BOUND_ZERO);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, BOUND_ZERO);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the 64 lanes in a fixed order: an inclusive scan inside each
// 16-lane row (shifts 1, 2, 4, 8), then the row totals are carried with the
// row broadcasts 15 and 31; lane 63 ends with the total (other lanes hold
// partial sums).
__device__ inline double wave_total_lane63(double v) {
  v += dpp_d<0x111, 0xf, true>(v);   // row_shr:1
  v += dpp_d<0x112, 0xf, true>(v);   // row_shr:2
  v += dpp_d<0x114, 0xf, true>(v);   // row_shr:4
  v += dpp_d<0x118, 0xf, true>(v);   // row_shr:8
  v += dpp_d<0x142, 0xa, false>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_d<0x143, 0xc, false>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// IRLS weight of a whitened residual: Huber min(1, c / |r|), or Tukey's
// biweight (1 - (r/c)^2)^2 inside c and 0 beyond.
template <typename T>
__device__ inline T huber_w(T r, T delta, bool tukey = false) {
  if (tukey) {
    const T t = r / delta, t2 = t * t;
    return t2 <= (T)1 ? ((T)1 - t2) * ((T)1 - t2) : (T)0;
  }
  const T a = fabs(r);
  return a <= delta ? (T)1 : delta / a;
}

// IRLS weight of the gradient edge between x_a and its right / lower neighbour x_b.
template <typename T>
__device__ inline T edge_weight(T xa, T xb, T g, T isd, T delta, bool tukey) {
  const T r = ((xb - xa) - g) * isd;
  return huber_w(r, delta, tukey) * isd * isd;
}

}  // namespace kf
