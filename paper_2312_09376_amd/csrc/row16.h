// Multiply-adds with a DPP row broadcast: a lane of each group of 16 hands its
// value to the group inside the instruction that uses it. Device code only.
#pragma once

#include <hip/hip_runtime.h>

#include "mma16.h"

namespace rbt {

// v of lane K of each group of 16 lanes, to the whole group.
template <int K>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + K, 0xF, 0xF, true));
}
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + K, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + K, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// x[j] += m * (y[j] of lane K of the group of 16), j = 0 .. N - 1. The
// broadcast is the first operand of v_fmac, a form that the compiler does not
// make for FP64 by itself (it moves both halves first); the leading s_nop is
// the distance that a DPP operand needs from the instruction that wrote it.
// dpp_distance(v): the same distance for a use of v by the compiler's own DPP.
#ifdef __AMDGCN__
template <typename C>
__device__ __forceinline__ void dpp_distance(C &v) {
  __asm__("s_nop 1" : "+v"(v));
}
// Values that are not needed any more (their registers become free).
template <int N, typename C>
__device__ __forceinline__ void forget(C (&v)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j) __asm__("" : "=v"(v[j]));
}
#define RBT_FMAC_OP(T, D, S0, M, K) \
  "v_fmac_" T "_dpp " D ", " S0 ", " M " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n\t"
#define RBT_FMAC_ROWS(C, T)                                                                     \
  template <int K, int N>                                                                       \
  __device__ __forceinline__ void fmac_rows(C *x, const C *y, C m) {                            \
    if constexpr (N >= 4) {                                                                     \
      __asm__("s_nop 1\n\t" RBT_FMAC_OP(T, "%0", "%4", "%8", "%9")                              \
                  RBT_FMAC_OP(T, "%1", "%5", "%8", "%9") RBT_FMAC_OP(T, "%2", "%6", "%8", "%9") \
                      RBT_FMAC_OP(T, "%3", "%7", "%8", "%9")                                    \
              : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3])                                  \
              : "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]), "v"(m), "n"(K));                    \
      fmac_rows<K, N - 4>(x + 4, y + 4, m);                                                     \
    } else if constexpr (N >= 2) {                                                              \
      __asm__("s_nop 1\n\t" RBT_FMAC_OP(T, "%0", "%2", "%4", "%5")                              \
                  RBT_FMAC_OP(T, "%1", "%3", "%4", "%5")                                        \
              : "+v"(x[0]), "+v"(x[1])                                                          \
              : "v"(y[0]), "v"(y[1]), "v"(m), "n"(K));                                          \
      fmac_rows<K, N - 2>(x + 2, y + 2, m);                                                     \
    } else if constexpr (N == 1) {                                                              \
      __asm__("s_nop 1\n\t" RBT_FMAC_OP(T, "%0", "%1", "%2", "%3")                              \
              : "+v"(x[0])                                                                      \
              : "v"(y[0]), "v"(m), "n"(K));                                                     \
    }                                                                                           \
  }                                                                                             \
  /* x[j] += m * (x[j] of lane K of the group), m of lane K zero */                             \
  template <int K, int N>                                                                       \
  __device__ __forceinline__ void fmac_rows(C *x, C m) {                                        \
    if constexpr (N >= 4) {                                                                     \
      __asm__("s_nop 1\n\t" RBT_FMAC_OP(T, "%0", "%0", "%4", "%5")                              \
                  RBT_FMAC_OP(T, "%1", "%1", "%4", "%5") RBT_FMAC_OP(T, "%2", "%2", "%4", "%5") \
                      RBT_FMAC_OP(T, "%3", "%3", "%4", "%5")                                    \
              : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3])                                  \
              : "v"(m), "n"(K));                                                                \
      fmac_rows<K, N - 4>(x + 4, m);                                                            \
    } else if constexpr (N >= 2) {                                                              \
      __asm__("s_nop 1\n\t" RBT_FMAC_OP(T, "%0", "%0", "%2", "%3")                              \
                  RBT_FMAC_OP(T, "%1", "%1", "%2", "%3")                                        \
              : "+v"(x[0]), "+v"(x[1])                                                          \
              : "v"(m), "n"(K));                                                                \
      fmac_rows<K, N - 2>(x + 2, m);                                                            \
    } else if constexpr (N == 1) {                                                              \
      __asm__("s_nop 1\n\t" RBT_FMAC_OP(T, "%0", "%0", "%1", "%2") : "+v"(x[0]) : "v"(m), "n"(K)); \
    }                                                                                           \
  }
RBT_FMAC_ROWS(double, "f64")
RBT_FMAC_ROWS(float, "f32")
#undef RBT_FMAC_ROWS
#undef RBT_FMAC_OP
#else  // the same in C++, for host builds of the kernels (tests)
template <typename C>
__device__ __forceinline__ void dpp_distance(C &) {}
template <int N, typename C>
__device__ __forceinline__ void forget(C (&)[N]) {}
template <int K, int N, typename C>
__device__ __forceinline__ void fmac_rows(C *x, const C *y, C m) {
  for (int j = 0; j < N; ++j) x[j] = fma_c(row_bcast<K>(y[j]), m, x[j]);
}
template <int K, int N, typename C>
__device__ __forceinline__ void fmac_rows(C *x, C m) {
  fmac_rows<K, N>(x, x, m);
}
#endif

}  // namespace rbt
