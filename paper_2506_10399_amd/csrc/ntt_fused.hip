// Base conversions fused with the transforms around them.
//
// ModUp, ModDown and the rescales all run: inverse NTT of a few limbs, an elementwise map from
// those limbs' coefficients to the coefficients of many limbs, forward NTT of these.  A transform
// is a row pass and a column pass (ntt.hip), the inverse one ends and the forward one begins with
// its column pass, and the map works coefficient by coefficient: so one kernel (k_mid) takes 16
// columns of the source limbs through the inverse column pass, keeps their coefficients in
// registers and, for each destination limb, maps them and runs the forward column pass.  The
// conversion's output is written once, half transformed, instead of written in coefficient form,
// read, and written again.  The inverse row pass before it reads the sources where they lie
// (k_inv_rows: no gathered copy), and ModDown's last step, elementwise as well, is taken by the
// forward row pass after it (k_fwd_rows_final).
//
// What bounds them: k_mid the vector ALU at large batches (a destination limb's coefficient takes 48
// instructions in fp64, 111 in integers), the row passes memory.  Measured at N = 2^16, 13 ciphertexts
// at level 4 with two special primes: ModUp's k_mid 82 us, where the inverse column pass, the
// conversion and the forward column pass took 22, 42 and 40; ModDown's 79 us for 22, 32 and 40, the
// row pass with the last step 65 us for 39 and 49.
#include <algorithm>

#include "ks_common.h"
#include "ntt_dev.h"
#include "ntt_fused.h"

namespace ficgcn {

// ---- inverse row pass, out of place --------------------------------------------------------
struct ModUpSrc {
  const uint64_t* const* srcs;   // or null: `one`
  const uint64_t* one;
  uint64_t* tmp;                 // [U][l1][N]
  uint64_t* D;                   // [U][nd][ext][N]: receives each digit's own limbs as they are
  int l1, nd, ext, alpha;
  __device__ __forceinline__ int mod(int i) const { return i; }
  __device__ __forceinline__ const uint64_t* in(int i, int u, int log_n) const {
    return (srcs ? (const uint64_t*)gld((const uint64_t*)(srcs + u)) : one) + ((size_t)i << log_n);
  }
  __device__ __forceinline__ uint64_t* out(int i, int u, int log_n) const {
    return tmp + (((size_t)u * l1 + i) << log_n);
  }
  __device__ __forceinline__ uint64_t* copy(int i, int u, int log_n) const {
    return D + ((((size_t)u * nd + i / alpha) * ext + i) << log_n);
  }
};

// the last nl limbs of both components of a ciphertext at `lvl`
struct LastSrc {
  uint64_t* const* cts;          // or null: `one`
  uint64_t* one;
  uint64_t* last;                // [2n][nl][N]
  int lvl, nl;
  __device__ __forceinline__ int mod(int t) const { return lvl - nl + 1 + t; }
  __device__ __forceinline__ const uint64_t* in(int t, int z, int log_n) const {
    const uint64_t* ct = cts ? (const uint64_t*)gld((const uint64_t*)(cts + (z >> 1))) : one;
    return ct + (((size_t)(z & 1) * (lvl + 1) + lvl - nl + 1 + t) << log_n);
  }
  __device__ __forceinline__ uint64_t* out(int t, int z, int log_n) const {
    return last + (((size_t)z * nl + t) << log_n);
  }
  __device__ __forceinline__ uint64_t* copy(int, int, int) const { return nullptr; }
};

template <int LOGC, bool FP, class S>
__device__ __forceinline__ void inv_rows_body(uint64_t* s, const S& src, int limb, int poly, const Tw& t, int log_n) {
  constexpr int COLS = row_cols<LOGC>();
  typedef PassGeo<LOGC, COLS> G;
  const Place<LOGC, COLS, true> p(threadIdx.x, blockIdx.x);
  const uint64_t* a = src.in(limb, poly, log_n);
  uint64_t* o = src.out(limb, poly, log_n);
  uint64_t* cp = src.copy(limb, poly, log_n);
  uint64_t x[G::EPT];
#pragma unroll
  for (int u = 0; u < G::EPT; ++u) x[u] = gld(a + p.gidx(p.r + G::TPC * u, log_n));
#pragma unroll
  for (int u = 0; u < G::EPT; ++u) {
    if (cp) gst(cp + p.gidx(p.r + G::TPC * u, log_n), x[u]);
    s[p.sidx(p.r + G::TPC * u)] = x[u];
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < G::EPT; ++v) {
    x[v] = s[p.sidx(p.r * G::EPT + v)];
    if (FP) x[v] = to_fbits(x[v]);
  }
  __syncthreads();
  inv_core<LOGC, COLS, true, FP>(x, s, p, t, log_n);
#pragma unroll
  for (int u = 0; u < G::EPT; ++u) gst(o + p.gidx(p.r + G::TPC * u, log_n), x[u]);
}

template <int LOGC, class S>
__global__ __launch_bounds__(64) void k_inv_rows(S src, int log_n, const uint64_t* __restrict__ tw,
                                                 const uint64_t* __restrict__ tws, const double* __restrict__ twf,
                                                 const Mod* __restrict__ mods) {
  typedef PassGeo<LOGC, row_cols<LOGC>()> G;
  __shared__ uint64_t s[G::LDS_WORDS];
  const int limb = blockIdx.y, poly = blockIdx.z;
  const int mi = src.mod(limb);
  const Mod md = cld(mods + mi);
  const uint64_t q = md.q;
  const Tw t = make_tw(tw, tws, twf, q, md.qinv, mi, log_n);
  if (fp_prime(q))
    inv_rows_body<LOGC, true>(s, src, limb, poly, t, log_n);
  else
    inv_rows_body<LOGC, false>(s, src, limb, poly, t, log_n);
}

// ---- inverse column pass, map, forward column pass -------------------------------------------
// A map takes the source limbs' coefficients (scaled, in [0, modulus)) to a destination's in the
// form that the forward stages take: a double in (-q, q), or a word in [0, 8q).  Its constants are
// entries of tables made with the context: a block's next entry arrives by a scalar load while the
// transform before it runs.
//
// The stages are ntt_dev.h's eight-point column stages.
enum MidKind { MID_UP, MID_DOWN, MID_RS, MID_RS2 };

// Coefficients y of the sources (each in [0, its prime)) -> one destination's (d.a holds, by kind):
//   MID_UP   fast base conversion, sum_t y_t h_t: h[2], their Shoup companions [2]
//   MID_DOWN the same less floor(P/2): + [1]
//   MID_RS   h - y, h = floor(q_l / 2), for y = [x + h]_{q_l}: h
//   MID_RS2  ((h1 - y_l) / q_l + h2 - y_{l-1}) / q_{l-1}: h1, h2, 1 / q_l and 1 / q_{l-1} with companions
// The chain descends, so a rescale's y lies below every destination prime.
template <int KIND, int NS, bool FP>
__device__ __forceinline__ uint64_t mid_map(const uint64_t (&y)[NS], int ns, const MidDst& d, bool src_fp, const Tw& t) {
  if (KIND == MID_UP || KIND == MID_DOWN) {
    if (FP && KIND == MID_UP && src_fp) {
      // every y_t < 2^50 < 2q: at most two signed products, each in (-5q/4, 5q/4)
      double a = fmulmod_s(b2f(to_fbits(y[0])), (double)d.a[0], t.qd, t.qinv);
      if (NS > 1 && ns > 1) a += fmulmod_s(b2f(to_fbits(y[NS - 1])), (double)d.a[1], t.qd, t.qinv);
      return f2b(sred(a, t.qd, t.qinv));
    }
    uint64_t a = mul_shoup_lazy4(y[0], d.a[0], d.a[2], t.c);
    if (NS > 1 && ns > 1) a += mul_shoup_lazy4(y[NS - 1], d.a[1], d.a[3], t.c);   // below 8q
    if (!FP && KIND == MID_UP) return a;
    a = csub(a, t.c.q4, t.c.nq4);
    if (FP) return f2b(sred(b2f(to_fbits(a)) - (double)d.a[4], t.qd, t.qinv));
    return a + (t.q - d.a[4]);
  }
  if (KIND == MID_RS) return FP ? f2b((double)d.a[0] - b2f(to_fbits(y[0]))) : sub_mod(d.a[0], y[0], t.q);
  if (FP) {
    const double u = (double)d.a[0] - b2f(to_fbits(y[NS - 1])), e = (double)d.a[1] - b2f(to_fbits(y[0]));
    const double v = sred(fmulmod_s(u, (double)d.a[2], t.qd, t.qinv) + e, t.qd, t.qinv);
    return f2b(fmulmod_s(v, (double)d.a[4], t.qd, t.qinv));
  }
  const uint64_t u = sub_mod(d.a[0], y[NS - 1], t.q), e = sub_mod(d.a[1], y[0], t.q);
  return mul_shoup(add_mod(mul_shoup(u, d.a[2], d.a[3], t.q), e, t.q), d.a[4], d.a[5], t.q);
}

struct MidArgs {
  const MidSrc* st;        // two sources a digit (one for MID_RS)
  const MidDst* dt;        // n_all destinations' room a digit
  const uint64_t* src;     // source limb t of digit d of polynomial z at src + z src_poly + (d src_digit + t) N
  uint64_t* dst;           // destination limb pos at dst + z dst_poly + (d dst_digit + pos) N
  size_t src_poly, dst_poly;   // words
  int src_digit, dst_digit;    // limbs
  int digits, ns, ns_last;     // sources of a digit, and of the last one
  int n_all;                   // a digit's sources and destinations (MID_UP), or its destinations
  int n_split;
};

// one source limb's columns to the map's input, in [0, modulus)
template <int LOGC, bool FP>
__device__ __forceinline__ void mid_source(uint64_t (&y)[8], uint64_t* s, const MidPlace<LOGC>& p, const Tw& t,
                                           const MidSrc& m, const uint64_t* a, int log_n) {
  const uint32_t w = p.word(log_n);
#pragma unroll
  for (int v = 0; v < 8; ++v) y[v] = (a + p.row(v, log_n))[w];
  mid_inv<LOGC, FP>(y, s, p, t);
  const double cd = (double)m.c;
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    const uint64_t x = FP ? from_fbits(f2b(fmulmod(b2f(y[v]), cd, t.qd, t.qinv))) : mul_shoup(y[v], m.c, m.cs, t.q);
    y[v] = add_mod(x, m.sh, t.q);
  }
}

template <int LOGC, int KIND, int NS, bool FP>
__device__ __forceinline__ void mid_dest(const uint64_t (&y)[NS][8], uint64_t* s, const MidPlace<LOGC>& p, const Tw& t,
                                         int ns, const MidDst& d, bool src_fp, uint64_t* o, int log_n) {
  MidTw<FP> first;
  if (FP) mid_fwd_first<LOGC, FP>(first, p, t);
  uint64_t x[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    uint64_t yy[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) yy[i] = y[i][u];
    x[u] = mid_map<KIND, NS, FP>(yy, ns, d, src_fp, t);
  }
  mid_fwd<LOGC, FP>(x, s, p, t, first);
  const uint32_t w = p.word(log_n);
#pragma unroll
  for (int v = 0; v < 8; ++v) (o + p.row(v, log_n))[w] = x[v];
}

// grid: (columns / 16, digits * n_split, polynomials); a block takes the n_split-th part of the
// destination limbs (small batches: more blocks, each repeating the sources' inverse pass)
template <int LOGC, int KIND, int NS>
__global__ __launch_bounds__((1 << LOGC) / 8 * MID_COLS) __attribute__((amdgpu_waves_per_eu(4))) void k_mid(
    const MidArgs m, TwTables tt, int log_n) {
  typedef MidGeo<LOGC> G;
  __shared__ uint64_t sb[2][G::BUF];
  const MidPlace<LOGC> p(threadIdx.x, blockIdx.x);
  const int digit = blockIdx.y / m.n_split, sl = blockIdx.y % m.n_split;
  const int ns = digit == m.digits - 1 ? m.ns_last : m.ns;
  const int n_dst = KIND == MID_UP ? m.n_all - ns : m.n_all;
  int k = n_dst * sl / m.n_split;
  const int k1 = n_dst * (sl + 1) / m.n_split;
  if (k >= k1) return;
  const MidDst* dt = m.dt + (size_t)digit * m.n_all;
  MidDst next = cld(dt + k);
  uint64_t y[NS][8];
  bool src_fp = true;
  int buf = 0;
  {
    const MidSrc* st = m.st + (size_t)digit * 2;
    const uint64_t* a = m.src + blockIdx.z * m.src_poly + ((size_t)(digit * m.src_digit) << log_n);
#pragma unroll
    for (int u = 0; u < NS; ++u)
      if (u < ns) {
        const MidSrc ms = cld(st + u);
        const Tw t = make_tw(tt.ipsi, tt.ipsi_s, tt.ipsi_f, ms.q, ms.qinv, ms.mi, log_n);
        const bool fp = fp_prime(ms.q);
        src_fp = src_fp && fp;
        if (fp)
          mid_source<LOGC, true>(y[u], sb[buf], p, t, ms, a + ((size_t)u << log_n), log_n);
        else
          mid_source<LOGC, false>(y[u], sb[buf], p, t, ms, a + ((size_t)u << log_n), log_n);
        buf ^= 1;
      }
    if (KIND == MID_RS2) {
      // limb l-1 after the first rescale, plus its half: (x_{l-1} + h_l - y_l) / q_l + floor(q_{l-1} / 2)
      const MidSrc ms = cld(st);
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const uint64_t d = sub_mod(ms.e[0], y[NS - 1][v], ms.q);
        y[0][v] = add_mod(mul_shoup(add_mod(y[0][v], d, ms.q), ms.e[1], ms.e[2], ms.q), ms.q / 2, ms.q);
      }
    }
  }
  uint64_t* const o = m.dst + blockIdx.z * m.dst_poly + ((size_t)(digit * m.dst_digit) << log_n);
#pragma unroll 1
  for (; k < k1; ++k) {
    const MidDst d = next;
    if (k + 1 < k1) next = cld(dt + k + 1);
    const Tw t = make_tw(tt.psi, tt.psi_s, tt.psi_f, d.q, d.qinv, d.mi, log_n);
    // y in its one form across the loop: nothing derived from it is kept in registers of its own
#pragma unroll
    for (int u = 0; u < NS; ++u)
#pragma unroll
      for (int v = 0; v < 8; ++v) asm volatile("" : "+v"(y[u][v]));
    uint64_t* const od = o + ((size_t)d.pos << log_n);
    if (fp_prime(d.q))
      mid_dest<LOGC, KIND, NS, true>(y, sb[buf], p, t, ns, d, src_fp, od, log_n);
    else
      mid_dest<LOGC, KIND, NS, false>(y, sb[buf], p, t, ns, d, src_fp, od, log_n);
    buf ^= 1;
  }
}

// ---- forward row pass with ModDown's last step ---------------------------------------------
template <int LOGC, bool FP>
__device__ __forceinline__ void fwd_rows_final_body(uint64_t* s, const uint64_t* conv, const uint64_t* acc,
                                                    const Tw& t, uint64_t pinv, uint64_t pinv_s, uint64_t* out,
                                                    const uint64_t* add, uint64_t g, bool accumulate, int log_n) {
  constexpr int COLS = row_cols<LOGC>();
  typedef PassGeo<LOGC, COLS> G;
  const Place<LOGC, COLS, true> p(threadIdx.x, blockIdx.x);
  uint64_t x[G::EPT];
#pragma unroll
  for (int u = 0; u < G::EPT; ++u) x[u] = conv[p.gidx(p.r + G::TPC * u, log_n)];
  fwd_core<LOGC, COLS, true, FP>(x, s, p, t, log_n);
  __syncthreads();
#pragma unroll
  for (int v = 0; v < G::EPT; ++v) s[p.sidx(p.r * G::EPT + v)] = x[v];
  __syncthreads();
  const double pd = (double)pinv;
#pragma unroll
  for (int u = 0; u < G::EPT; ++u) {
    const size_t n = p.gidx(p.r + G::TPC * u, log_n);
    const uint64_t w = s[p.sidx(p.r + G::TPC * u)], a = acc[n];
    uint64_t v;
    if (FP)   // acc in [0, q), the transform in (-q, q)
      v = from_fbits(f2b(canon(fmulmod_s(sred(b2f(to_fbits(a)) - b2f(w), t.qd, t.qinv), pd, t.qd, t.qinv), t.qd)));
    else
      v = mul_shoup(sub_mod(a, canon8(w, t.c, t.q), t.q), pinv, pinv_s, t.q);
    if (add) v = add_mod(v, gld(add + (g == 1 ? (uint32_t)n : auto_idx((uint32_t)n, g, log_n))), t.q);
    if (accumulate) v = add_mod(v, gld(out + n), t.q);
    gst(out + n, v);
  }
}

template <int LOGC>
__global__ __launch_bounds__(64) void k_fwd_rows_final(const uint64_t* __restrict__ acc, const uint64_t* __restrict__ conv,
                                                       int ext, int l1, MDK k, const FinalJob* __restrict__ jobs,
                                                       FinalJob one, TwTables tt, int log_n) {
  typedef PassGeo<LOGC, row_cols<LOGC>()> G;
  __shared__ uint64_t s[G::LDS_WORDS];
  const int i = blockIdx.y, z = blockIdx.z, comp = z & 1;
  const FinalJob jb = jobs ? jobs[z >> 1] : one;
  const Mod md = cld(tt.mods + i);
  const uint64_t q = md.q;
  const Tw t = make_tw(tt.psi, tt.psi_s, tt.psi_f, q, md.qinv, i, log_n);
  const uint64_t* a = acc + (((size_t)z * ext + i) << log_n);
  const uint64_t* cv = conv + (((size_t)z * l1 + i) << log_n);
  uint64_t* out = jb.out + (((size_t)comp * l1 + i) << log_n);
  const uint64_t* add = comp ? jb.add1 : jb.add0;
  if (add) add += (size_t)i << log_n;
  const uint64_t g = comp ? 1 : jb.g;
  if (fp_prime(q))
    fwd_rows_final_body<LOGC, true>(s, cv, a, t, k.pinv[i], k.pinv_s[i], out, add, g, jb.accumulate, log_n);
  else
    fwd_rows_final_body<LOGC, false>(s, cv, a, t, k.pinv[i], k.pinv_s[i], out, add, g, jb.accumulate, log_n);
}

// ---- launches ------------------------------------------------------------------------------
#define BY_LOGC_ROW(lc, X)                                       \
  switch (lc) {                                                  \
    case 4: X(4); break;                                         \
    case 5: X(5); break;                                         \
    case 6: X(6); break;                                         \
    case 7: X(7); break;                                         \
    case 8: X(8); break;                                         \
    case 9: X(9); break;                                         \
    default: FICGCN_THROW(EINVAL_, "unsupported ring degree");   \
  }
#define BY_LOGC_MID(lc, X)                                       \
  switch (lc) {                                                  \
    case 4: X(4); break;                                         \
    case 5: X(5); break;                                         \
    case 6: X(6); break;                                         \
    case 7: X(7); break;                                         \
    case 8: X(8); break;                                         \
    default: FICGCN_THROW(EINVAL_, "unsupported ring degree");   \
  }

template <class S>
static void inv_rows(ckks_ctx* c, const S& src, int n_limbs, int n_polys) {
  const int lr = c->log_n - ntt_mid_log(c);
  const TwTables tt = tw_tables(c);
#define X(LC)                                                                                                       \
  hipLaunchKernelGGL((k_inv_rows<LC, S>), dim3((c->N >> LC) / row_cols<LC>(), n_limbs, n_polys), dim3(64), 0,       \
                     c->stream, src, c->log_n, tt.ipsi, tt.ipsi_s, tt.ipsi_f, tt.mods)
  BY_LOGC_ROW(lr, X)
#undef X
  HIPCHECK(hipGetLastError());
}

// parts the destination limbs are taken in: at least ~1024 blocks where the limbs allow it
static int mid_split(ckks_ctx* c, int lc, int digits, int n_polys, int n_dst) {
  const size_t blocks = (size_t)((c->N >> lc) / MID_COLS) * digits * n_polys;
  return (int)std::min<size_t>(n_dst, std::max<size_t>(1, (1024 + blocks - 1) / blocks));
}

template <int KIND, int NS>
static void mid(ckks_ctx* c, MidArgs m, int n_polys, int most) {
  const int lc = ntt_mid_log(c);
  const TwTables tt = tw_tables(c);
  m.n_split = mid_split(c, lc, m.digits, n_polys, most);
#define X(LC)                                                                                                 \
  hipLaunchKernelGGL((k_mid<LC, KIND, NS>), dim3((c->N >> LC) / MID_COLS, m.digits * m.n_split, n_polys),     \
                     dim3((1 << LC) / 8 * MID_COLS), 0, c->stream, m, tt, c->log_n)
  BY_LOGC_MID(lc, X)
#undef X
  HIPCHECK(hipGetLastError());
}

void modup_polys(ckks_ctx* c, int level, const uint64_t* const* srcs, const uint64_t* one, int U, uint64_t* tmp,
                 uint64_t* D) {
  const size_t N = c->N;
  const int a = c->alpha, l1 = level + 1, ext = l1 + a;
  const int nd = (l1 + a - 1) / a;
  inv_rows(c, ModUpSrc{srcs, one, tmp, D, l1, nd, ext, a}, l1, U);
  const MidLevel& ml = c->mid[level];
  const MidArgs m{c->mid_src + ml.up_s, c->mid_dst + ml.up_d, tmp, D, l1 * N, nd * ext * N, a, ext, nd, a,
                  l1 - (nd - 1) * a, ext, 1};
  if (a == 1)
    mid<MID_UP, 1>(c, m, U, ext - 1);
  else
    mid<MID_UP, 2>(c, m, U, ext - 1);
  // every extended limb to evaluation form except each digit's own limbs
  ntt_fwd_rows(c, D, ext, lm_ext(level, c->L), U * nd, (size_t)ext * N, a, l1);
}

void moddown_polys(ckks_ctx* c, int level, uint64_t* acc, int Z, uint64_t* conv, bool rows) {
  const size_t N = c->N;
  const int a = c->alpha, l1 = level + 1, ext = l1 + a;
  ntt_inv_rows(c, acc + (size_t)l1 * N, a, LimbMap{c->L, 1 << 30, 0}, Z, (size_t)ext * N);
  const MidLevel& ml = c->mid[level];
  const MidArgs m{c->mid_src + ml.down_s, c->mid_dst + ml.down_d, acc + (size_t)l1 * N, conv, ext * N, l1 * N, 0, 0, 1,
                  a, a, l1, 1};
  if (a == 1)
    mid<MID_DOWN, 1>(c, m, Z, l1);
  else
    mid<MID_DOWN, 2>(c, m, Z, l1);
  if (rows) ntt_fwd_rows(c, conv, l1, lm_q(l1), Z, (size_t)l1 * N);
}

void moddown_final(ckks_ctx* c, int level, const uint64_t* acc, uint64_t* conv, const FinalJob* jobs,
                   const FinalJob& one, int n) {
  const int l1 = level + 1, ext = l1 + c->alpha;
  const int lr = c->log_n - ntt_mid_log(c);
  const TwTables tt = tw_tables(c);
  const MDK& k = c->mdk[level];
#define X(LC)                                                                                                    \
  hipLaunchKernelGGL(k_fwd_rows_final<LC>, dim3((c->N >> LC) / row_cols<LC>(), l1, 2 * n), dim3(64), 0,          \
                     c->stream, acc, conv, ext, l1, k, jobs, one, tt, c->log_n)
  BY_LOGC_ROW(lr, X)
#undef X
  HIPCHECK(hipGetLastError());
}

void rescale_prep(ckks_ctx* c, int level, uint64_t* const* cts, uint64_t* one, int n, uint64_t* last, uint64_t* d) {
  const size_t N = c->N;
  inv_rows(c, LastSrc{cts, one, last, level, 1}, 1, 2 * n);
  const MidLevel& ml = c->mid[level];
  const MidArgs m{c->mid_src + ml.rs_s, c->mid_dst + ml.rs_d, last, d, N, level * N, 0, 0, 1, 1, 1, level, 1};
  mid<MID_RS, 1>(c, m, 2 * n, level);
  ntt_fwd_rows(c, d, level, lm_q(level), 2 * n, level * N);
}

void rescale2_prep(ckks_ctx* c, int level, uint64_t* const* cts, int n, uint64_t* last, uint64_t* f) {
  const size_t N = c->N;
  inv_rows(c, LastSrc{cts, nullptr, last, level, 2}, 2, 2 * n);
  const MidLevel& ml = c->mid[level];
  const MidArgs m{c->mid_src + ml.rs2_s, c->mid_dst + ml.rs2_d, last, f, 2 * N, (level - 1) * N, 0, 0, 1, 2, 2,
                  level - 1, 1};
  mid<MID_RS2, 2>(c, m, 2 * n, level - 1);
  ntt_fwd_rows(c, f, level - 1, lm_q(level - 1), 2 * n, (level - 1) * N);
}

}  // namespace ficgcn
