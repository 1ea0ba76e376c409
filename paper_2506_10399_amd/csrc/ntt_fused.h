// Transforms fused with the base conversions of ModUp, ModDown and the rescales (ntt_fused.hip).
#pragma once
#include "internal.h"

namespace ficgcn {

// ModUp and ModDown go through the fused kernels for one or two special primes (every shipped
// configuration): a thread holds eight coefficients of each of a digit's limbs, the tables have room for
// two sources a digit, and a sum of two lazy products stays below 8q.  Longer digits take the separate passes.
inline bool fused_basis(const ckks_ctx* c) { return c->alpha <= 2; }
// ModUp of U polynomials [l1][N] in evaluation form, poly u at srcs[u] (device table) or, when
// srcs is null, at `one` (U = 1): D [U][nd][ext][N].  tmp: U * l1 limbs.
void modup_polys(ckks_ctx* c, int level, const uint64_t* const* srcs, const uint64_t* one, int U, uint64_t* tmp,
                 uint64_t* D);
// ModDown's conversion of Z accumulators [ext][N] (poly z at acc + z * ext * N; their P limbs are
// left half transformed, after the inverse row pass): conv [Z][l1][N].  The transform of conv stops before its row pass
// when `rows` is false (a row pass with a fused final step follows).
void moddown_polys(ckks_ctx* c, int level, uint64_t* acc, int Z, uint64_t* conv, bool rows);
// One final step per ciphertext on ModDown's conversion before its row pass (moddown_polys with
// rows = false): the row pass, then outs (+)= ((acc - conv) P^-1 + add).
struct FinalJob {
  uint64_t* out;          // [2][l1][N]
  const uint64_t* add0;   // [l1][N] or null, read through sigma_g
  const uint64_t* add1;   // [l1][N] or null
  uint64_t g;
  int32_t accumulate;
  int32_t pad;
};
// jobs: device table of n entries, or null with `one` (n = 1); acc [n][2][ext][N]; conv is scratch
void moddown_final(ckks_ctx* c, int level, const uint64_t* acc, uint64_t* conv, const FinalJob* jobs,
                   const FinalJob& one, int n);
// Rescale corrections of n ciphertexts at `level`, ciphertext i at cts[i] (device table) or, when cts
// is null, `one` (n = 1): last: 2n limbs, d: [2n][level][N] in evaluation form
void rescale_prep(ckks_ctx* c, int level, uint64_t* const* cts, uint64_t* one, int n, uint64_t* last, uint64_t* d);
// two rescales: last: 4n limbs, f: [2n][level-1][N]
void rescale2_prep(ckks_ctx* c, int level, uint64_t* const* cts, int n, uint64_t* last, uint64_t* f);

}  // namespace ficgcn
