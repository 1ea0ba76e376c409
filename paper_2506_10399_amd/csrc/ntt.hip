// Negacyclic NTT over Z_q[X]/(X^N + 1) for gfx950.
//
// Forward transform (Cooley-Tukey, twiddles psi^{brev(m+i)} merged with the
// negacyclic twist): coefficients in natural order -> evaluations at the odd
// powers psi^{2 brev(k) + 1} in bit-reversed order k.  Inverse: the
// Gentleman-Sande mirror, then a multiply by N^{-1}.
//
// A limb of N = 2^16 words (512 KiB) exceeds the LDS, so each transform runs
// as two passes of N = N1 * N2:
//   column pass: the stages m < N1 touch only the N1 elements j0 + k*N2 of one
//                column j0 (a C = N1-point sub-transform);
//   row pass   : the stages m >= N1 stay inside one contiguous chunk of C = N2
//                words.
// Inside a pass, TPC = 2^floor(log C / 2) threads share one sub-transform and
// each holds EPT = C / TPC elements in registers:
//   strided layout     thread r holds elements r + TPC*u  (u < EPT): the
//                      stages with butterfly distance t >= TPC are local;
//   contiguous layout  thread r holds elements r*EPT + v (v < EPT): the stages
//                      with t < TPC are local.
// One LDS transpose switches layouts (a second one in the row pass keeps the
// global loads and stores coalesced).  Every twiddle a thread needs is read
// before its stages run.  A workgroup handles COLS columns (column pass) or
// chunks (row pass); COLS is picked per ring degree by the autotuner.
// The stages themselves are in ntt_dev.h.
// For the 50-bit Q primes (fp64 residue arithmetic, fpmod.h) the limb travels
// between the two passes as the bit patterns of its doubles: the first pass
// converts on load, the second on store.
#include <algorithm>

#include "ntt_dev.h"

namespace ficgcn {

// ModUp output: digit d of a source owns limbs d*alpha .. d*alpha+alpha-1, which
// hold evaluation-form input already; polys run digit-fastest over sources
__device__ __forceinline__ bool skip_limb(int limb, int poly, int skip_alpha, int skip_q) {
  return skip_alpha > 0 && limb < skip_q && limb / skip_alpha == poly % ((skip_q + skip_alpha - 1) / skip_alpha);
}

// One pass over one sub-transform set of a limb; FP selects the fp64 residue arithmetic.
template <int LOGC, int COLS, bool INV, bool ROW, bool FP>
__device__ __forceinline__ void ntt_pass_body(uint64_t* s, uint64_t* a, const Tw& t, int log_n, int mi,
                                              const uint64_t* __restrict__ ninv,
                                              const uint64_t* __restrict__ ninv_s) {
  typedef PassGeo<LOGC, COLS> G;
  constexpr int TPC = G::TPC, EPT = G::EPT;
  const Place<LOGC, COLS, ROW> p(threadIdx.x, blockIdx.x);
  uint64_t x[EPT];
  if (!INV) {
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      x[u] = a[p.gidx(p.r + TPC * u, log_n)];
      if (FP && !ROW) x[u] = to_fbits(x[u]);
    }
    fwd_core<LOGC, COLS, ROW, FP>(x, s, p, t, log_n);
    if (ROW) {
      // residues, back in the strided layout for a coalesced store
#pragma unroll
      for (int v = 0; v < EPT; ++v) x[v] = FP ? from_fbits(f2b(canon(b2f(x[v]), t.qd))) : canon8(x[v], t.c, t.q);
      __syncthreads();
#pragma unroll
      for (int v = 0; v < EPT; ++v) s[p.sidx(p.r * EPT + v)] = x[v];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < EPT; ++u) a[p.gidx(p.r + TPC * u, log_n)] = s[p.sidx(p.r + TPC * u)];
    } else {
#pragma unroll
      for (int v = 0; v < EPT; ++v) a[p.gidx(p.r * EPT + v, log_n)] = x[v];
    }
  } else {
    if (ROW) {
      // coalesced load, then the contiguous layout
#pragma unroll
      for (int u = 0; u < EPT; ++u) s[p.sidx(p.r + TPC * u)] = a[p.gidx(p.r + TPC * u, log_n)];
      __syncthreads();
#pragma unroll
      for (int v = 0; v < EPT; ++v) {
        x[v] = s[p.sidx(p.r * EPT + v)];
        if (FP) x[v] = to_fbits(x[v]);
      }
      __syncthreads();
    } else {
#pragma unroll
      for (int v = 0; v < EPT; ++v) x[v] = a[p.gidx(p.r * EPT + v, log_n)];
    }
    inv_core<LOGC, COLS, ROW, FP>(x, s, p, t, log_n);
    if (!ROW) {
      const uint64_t ni = ninv[mi], nis = ninv_s[mi];
      const double nid = (double)ni;
#pragma unroll
      for (int u = 0; u < EPT; ++u)
        x[u] = FP ? from_fbits(f2b(fmulmod(b2f(x[u]), nid, t.qd, t.qinv))) : mul_shoup(x[u], ni, nis, t.q);
    }
#pragma unroll
    for (int u = 0; u < EPT; ++u) a[p.gidx(p.r + TPC * u, log_n)] = x[u];
  }
}

// ROW: row pass (sub-transform = contiguous chunk), else column pass.
template <int LOGC, int COLS, bool INV, bool ROW>
__global__ __launch_bounds__((1 << (LOGC / 2)) * COLS) void k_ntt_pass(
    uint64_t* __restrict__ base, int log_n, LimbMap map, size_t poly_stride, const uint64_t* __restrict__ tw,
    const uint64_t* __restrict__ tws, const double* __restrict__ twf, const Mod* __restrict__ mods,
    const uint64_t* __restrict__ ninv, const uint64_t* __restrict__ ninv_s, int skip_alpha, int skip_q) {
  __shared__ uint64_t s[PassGeo<LOGC, COLS>::LDS_WORDS];
  const int limb = blockIdx.y, poly = blockIdx.z;
  if (skip_limb(limb, poly, skip_alpha, skip_q)) return;
  const int mi = lm_mod(map, limb);
  const Mod m = cld(mods + mi);
  const uint64_t q = m.q;
  uint64_t* a = base + poly * poly_stride + ((size_t)limb << log_n);
  const Tw t = make_tw(tw, tws, twf, q, m.qinv, mi, log_n);
  if (fp_prime(q))
    ntt_pass_body<LOGC, COLS, INV, ROW, true>(s, a, t, log_n, mi, ninv, ninv_s);
  else
    ntt_pass_body<LOGC, COLS, INV, ROW, false>(s, a, t, log_n, mi, ninv, ninv_s);
}

// ---- launch selection --------------------------------------------------------
template <bool INV, bool ROW, int COLS>
static void launch_c(int logc, dim3 grid, hipStream_t st, uint64_t* base, int log_n, LimbMap map, size_t ps,
                     const Tables& t, int sa, int sq) {
  const uint64_t* tw = INV ? t.ipsi : t.psi;
  const uint64_t* tws = INV ? t.ipsi_s : t.psi_s;
  const double* twf = INV ? t.ipsi_f : t.psi_f;
  switch (logc) {
#define CASE(L)                                                                                                   \
  case L:                                                                                                         \
    hipLaunchKernelGGL((k_ntt_pass<L, COLS, INV, ROW>), grid, dim3((1 << (L / 2)) * COLS), 0, st, base, log_n, map, \
                       ps, tw, tws, twf, t.mods, t.ninv, t.ninv_s, sa, sq);                                       \
    break;
    CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9)
#undef CASE
    default: FICGCN_THROW(EINVAL_, "unsupported ring degree");
  }
}

template <bool INV, bool ROW>
static void launch(ckks_ctx* c, int logc, int cols, uint64_t* base, int n_limbs, LimbMap map, int n_polys,
                   size_t ps, int sa, int sq) {
  const int units = c->N >> logc;   // columns (column pass) or chunks (row pass)
  if (units % cols) cols = 1;
  dim3 grid(units / cols, n_limbs, n_polys);
  switch (cols) {
    case 1: launch_c<INV, ROW, 1>(logc, grid, c->stream, base, c->log_n, map, ps, c->t, sa, sq); break;
    case 2: launch_c<INV, ROW, 2>(logc, grid, c->stream, base, c->log_n, map, ps, c->t, sa, sq); break;
    case 4: launch_c<INV, ROW, 4>(logc, grid, c->stream, base, c->log_n, map, ps, c->t, sa, sq); break;
    case 8: launch_c<INV, ROW, 8>(logc, grid, c->stream, base, c->log_n, map, ps, c->t, sa, sq); break;
    default: launch_c<INV, ROW, 16>(logc, grid, c->stream, base, c->log_n, map, ps, c->t, sa, sq); break;
  }
}

// N = 2^l1 (column pass) * 2^l2 (row pass); each pass between 2^4 and 2^9 points
static void split(const ckks_ctx* c, int& l1, int& l2) {
  l1 = c->ntt_split ? c->ntt_split : c->log_n / 2;
  l2 = c->log_n - l1;
  if (l1 < 4 || l1 > 9 || l2 < 4 || l2 > 9) FICGCN_THROW(EINVAL_, "NTT split outside 2^4..2^9 points per pass");
}

void ntt_fwd(ckks_ctx* c, uint64_t* base, int n_limbs, LimbMap map, int n_polys, size_t poly_stride, int skip_alpha,
             int skip_q) {
  ProfScope ps(c, "ntt");
  if (n_limbs <= 0 || n_polys <= 0) return;
  int l1, l2;
  split(c, l1, l2);
  launch<false, false>(c, l1, c->ntt_cols[0], base, n_limbs, map, n_polys, poly_stride, skip_alpha, skip_q);
  launch<false, true>(c, l2, c->ntt_cols[1], base, n_limbs, map, n_polys, poly_stride, skip_alpha, skip_q);
  HIPCHECK(hipGetLastError());
}

void ntt_inv(ckks_ctx* c, uint64_t* base, int n_limbs, LimbMap map, int n_polys, size_t poly_stride) {
  ProfScope ps(c, "ntt");
  if (n_limbs <= 0 || n_polys <= 0) return;
  int l1, l2;
  split(c, l1, l2);
  launch<true, true>(c, l2, c->ntt_cols[1], base, n_limbs, map, n_polys, poly_stride, 0, 0);
  launch<true, false>(c, l1, c->ntt_cols[0], base, n_limbs, map, n_polys, poly_stride, 0, 0);
  HIPCHECK(hipGetLastError());
}

int ntt_mid_log(const ckks_ctx* c) {
  int l1, l2;
  split(c, l1, l2);
  return std::min(l1, 8);   // a fused column pass holds its sources' coefficients in registers
}

void ntt_fwd_rows(ckks_ctx* c, uint64_t* base, int n_limbs, LimbMap map, int n_polys, size_t poly_stride,
                  int skip_alpha, int skip_q) {
  ProfScope ps(c, "ntt");
  launch<false, true>(c, c->log_n - ntt_mid_log(c), c->ntt_cols[1], base, n_limbs, map, n_polys, poly_stride,
                      skip_alpha, skip_q);
  HIPCHECK(hipGetLastError());
}

void ntt_inv_rows(ckks_ctx* c, uint64_t* base, int n_limbs, LimbMap map, int n_polys, size_t poly_stride) {
  ProfScope ps(c, "ntt");
  launch<true, true>(c, c->log_n - ntt_mid_log(c), c->ntt_cols[1], base, n_limbs, map, n_polys, poly_stride, 0, 0);
  HIPCHECK(hipGetLastError());
}

}  // namespace ficgcn
