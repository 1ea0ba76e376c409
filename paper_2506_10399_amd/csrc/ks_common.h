// Small device helpers of the key-switching and ciphertext kernels.
#pragma once
#include "internal.h"

namespace ficgcn {

// Accesses through pointers read from device tables (job lists, term lists,
// pointer arrays).  The compiler cannot tell that such a pointer addresses
// global memory and would emit flat accesses, which also count on the
// scalar-load counter: every read of the next table entry would then wait for
// all vector loads in flight.  These pin the access to the global segment.
typedef __attribute__((address_space(1))) uint64_t gu64;
__device__ __forceinline__ uint64_t gld(const uint64_t* p) { return *(const gu64*)p; }
__device__ __forceinline__ void gst(uint64_t* p, uint64_t v) { *(gu64*)p = v; }

// a wave-uniform load from a table that no kernel writes while it is read: a scalar load
template <class T>
__device__ __forceinline__ T cld(const T* p) {
  static_assert(sizeof(T) % 8 == 0, "whole words");
  typedef const __attribute__((address_space(4))) uint64_t cu64;
  uint64_t w[sizeof(T) / 8];
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 8; ++i) w[i] = ((cu64*)p)[i];
  T r;
  __builtin_memcpy(&r, w, sizeof(T));
  return r;
}

__device__ __forceinline__ uint32_t auto_idx(uint32_t k, uint64_t g, int log_n) {
  // evaluation index k holds A(psi^(2 brev(k) + 1)); sigma_g reads the index of psi^(g (2 brev(k) + 1))
  uint32_t N2 = 2u << log_n;
  uint32_t e = 2u * bitrev(k, log_n) + 1u;
  uint32_t ge = (uint32_t)(((uint64_t)e * g) & (N2 - 1));
  return bitrev((ge - 1u) >> 1, log_n);
}

}  // namespace ficgcn
