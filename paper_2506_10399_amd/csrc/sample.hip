// Randomness, key generation and symmetric encryption on the device.
//
// Every random polynomial is read from a ChaCha20 stream (block function of
// RFC 8439): key words (seed mod 2^32, seed >> 32, 0, 0, 0, 0, 0, 0), a
// three-word nonce naming the stream, block counter 0, 1, ...  Coefficient j
//   uniform mod q : words 4j..4j+3 as a little-endian 128-bit integer, mod q
//   ternary       : x = words 2j, 2j+1 as a 64-bit integer, (x mod 3) - 1
//   CBD(21)       : popcount(x & (2^21-1)) - popcount((x >> 21) & (2^21-1))
// Streams: secret (1,0,0); key 'a' (2, tag, digit*65536 + prime index);
// key 'e' (3, tag, digit); ciphertext 'a' (4, id, prime index); ciphertext
// 'e' (5, id, 0).  A ciphertext's 'a' may be keyed by a public seed of its own
// (a seeded ciphertext: the server regenerates 'a' from that seed and the id).  A rotation key's tag is its Galois element, the
// relinearisation key's tag is 0.
#include <algorithm>

#include "ks_common.h"
#include "ntt_dev.h"

namespace ficgcn {

constexpr int SB = 256;

__device__ __forceinline__ uint32_t rotl(uint32_t x, int r) { return (x << r) | (x >> (32 - r)); }

__device__ __forceinline__ void qr(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) {
  a += b; d ^= a; d = rotl(d, 16);
  c += d; b ^= c; b = rotl(b, 12);
  a += b; d ^= a; d = rotl(d, 8);
  c += d; b ^= c; b = rotl(b, 7);
}

__device__ void chacha_block(uint64_t seed, uint32_t n0, uint32_t n1, uint32_t n2, uint32_t ctr, uint32_t out[16]) {
  uint32_t s[16] = {0x61707865u, 0x3320646eu, 0x79622d32u, 0x6b206574u, (uint32_t)seed, (uint32_t)(seed >> 32),
                    0, 0, 0, 0, 0, 0, ctr, n0, n1, n2};
  uint32_t x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = s[i];
#pragma unroll 1
  for (int r = 0; r < 10; ++r) {
    qr(x[0], x[4], x[8], x[12]); qr(x[1], x[5], x[9], x[13]); qr(x[2], x[6], x[10], x[14]); qr(x[3], x[7], x[11], x[15]);
    qr(x[0], x[5], x[10], x[15]); qr(x[1], x[6], x[11], x[12]); qr(x[2], x[7], x[8], x[13]); qr(x[3], x[4], x[9], x[14]);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) out[i] = x[i] + s[i];
}

// the coefficients of one block
__device__ __forceinline__ void uniform4(const uint32_t (&w)[16], const Mod& m, uint64_t (&v)[4]) {
#pragma unroll
  for (int u = 0; u < 4; ++u)
    v[u] = reduce128((uint64_t)w[4 * u + 2] | ((uint64_t)w[4 * u + 3] << 32),
                     (uint64_t)w[4 * u] | ((uint64_t)w[4 * u + 1] << 32), m);
}
// dist 0 = ternary, 1 = CBD(21)
__device__ __forceinline__ void small8(const uint32_t (&w)[16], int dist, int64_t (&v)[8]) {
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const uint64_t x = (uint64_t)w[2 * u] | ((uint64_t)w[2 * u + 1] << 32);
    if (dist == 0) {
      v[u] = (int64_t)(x % 3) - 1;
    } else {
      const uint64_t msk = (1ull << 21) - 1;
      v[u] = (int64_t)__popcll(x & msk) - (int64_t)__popcll((x >> 21) & msk);
    }
  }
}

// one thread = one block = 4 coefficients of one limb
__global__ void k_uniform(uint64_t* __restrict__ out, uint64_t seed, uint32_t kind, uint32_t a, uint32_t b0,
                          LimbMap map, int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const uint32_t blk = blockIdx.x * SB + threadIdx.x;
  if ((size_t)blk * 4 >= N) return;
  const int i = blockIdx.y;
  const int mi = lm_mod(map, i);
  uint32_t w[16];
  chacha_block(seed, kind, a, b0 + (uint32_t)mi, blk, w);
  const Mod m = mods[mi];
  uint64_t v[4];
  uniform4(w, m, v);
#pragma unroll
  for (int u = 0; u < 4; ++u) out[i * N + (size_t)blk * 4 + u] = v[u];
}

void sample_uniform(ckks_ctx* c, uint64_t* out, uint64_t seed, uint32_t kind, uint32_t a, uint32_t b0, int n_limbs,
                    LimbMap map, uint32_t) {
  int nb = (c->N / 4 + SB - 1) / SB;
  hipLaunchKernelGGL(k_uniform, dim3(nb, n_limbs), dim3(SB), 0, c->stream, out, seed, kind, a, b0, map, c->log_n,
                     c->t.mods);
  HIPCHECK(hipGetLastError());
}

// ---- bit-packed residues (transport of client words) ----
// A limb of N residues below 2^bits travels as N * bits / 64 words: residue r of the
// limb holds bits r * bits .. r * bits + bits - 1 of the limb's little-endian bit stream.
// count polynomials of n_limbs limbs: polynomial z's limbs at in + z * in_stride
// (resp. out + z * out_stride), limbs N (packed: N * bits / 64) words apart.

// one thread per packed word: the residues that overlap it, shifted into place
__global__ void k_pack(const uint64_t* __restrict__ in, size_t in_stride, uint64_t* __restrict__ out,
                       size_t out_stride, int bits, int log_n) {
  const size_t N = (size_t)1 << log_n;
  const size_t wpl = (N * (size_t)bits) >> 6;
  const size_t w = blockIdx.x * (size_t)SB + threadIdx.x;
  if (w >= wpl) return;
  const uint64_t* src = in + blockIdx.z * in_stride + (size_t)blockIdx.y * N;
  const uint64_t mask = bits == 64 ? ~0ull : (1ull << bits) - 1;
  const size_t b0 = w * 64;
  uint64_t v = 0;
  for (size_t r = b0 / bits; r < N && r * bits < b0 + 64; ++r) {
    const uint64_t x = src[r] & mask;
    const long long off = (long long)(r * bits) - (long long)b0;   // in (-bits, 64)
    v |= off >= 0 ? x << off : x >> (-off);
  }
  out[blockIdx.z * out_stride + (size_t)blockIdx.y * wpl + w] = v;
}

// one thread per residue: one or two packed words
__global__ void k_unpack(const uint64_t* __restrict__ in, size_t in_stride, uint64_t* __restrict__ out,
                         size_t out_stride, int bits, int log_n) {
  const size_t N = (size_t)1 << log_n;
  const size_t wpl = (N * (size_t)bits) >> 6;
  const size_t r = blockIdx.x * (size_t)SB + threadIdx.x;
  if (r >= N) return;
  const uint64_t* src = in + blockIdx.z * in_stride + (size_t)blockIdx.y * wpl;
  const size_t b = r * bits, w = b >> 6;
  const int sh = (int)(b & 63);
  uint64_t v = src[w] >> sh;
  if (sh + bits > 64) v |= src[w + 1] << (64 - sh);   // the residue's last bit lies in the limb
  const uint64_t mask = bits == 64 ? ~0ull : (1ull << bits) - 1;
  out[blockIdx.z * out_stride + (size_t)blockIdx.y * N + r] = v & mask;
}

void pack_residues(ckks_ctx* c, const uint64_t* in, size_t in_stride, uint64_t* out, size_t out_stride,
                   int n_limbs, size_t count, int bits, bool unpack) {
  const size_t N = c->N;
  const size_t wpl = (N * (size_t)bits) >> 6;
  const size_t units = unpack ? N : wpl;
  const int nb = (int)((units + SB - 1) / SB);
  constexpr size_t CHUNK = 4096;   // polynomials per launch (grid z)
  for (size_t z0 = 0; z0 < count; z0 += CHUNK) {
    const size_t nz = std::min(CHUNK, count - z0);
    if (unpack)
      hipLaunchKernelGGL(k_unpack, dim3(nb, n_limbs, (uint32_t)nz), dim3(SB), 0, c->stream, in + z0 * in_stride,
                         in_stride, out + z0 * out_stride, out_stride, bits, c->log_n);
    else
      hipLaunchKernelGGL(k_pack, dim3(nb, n_limbs, (uint32_t)nz), dim3(SB), 0, c->stream, in + z0 * in_stride,
                         in_stride, out + z0 * out_stride, out_stride, bits, c->log_n);
    HIPCHECK(hipGetLastError());
  }
}

// one thread = one block = 8 coefficients, written as residues of every limb
__global__ void k_small(uint64_t* __restrict__ out, uint64_t seed, uint32_t kind, uint32_t a, uint32_t b, int dist,
                        int n_limbs, LimbMap map, int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const uint32_t blk = blockIdx.x * SB + threadIdx.x;
  if ((size_t)blk * 8 >= N) return;
  uint32_t w[16];
  chacha_block(seed, kind, a, b, blk, w);
  int64_t v[8];
  small8(w, dist, v);
  for (int i = 0; i < n_limbs; ++i) {
    const uint64_t q = mods[lm_mod(map, i)].q;
#pragma unroll
    for (int u = 0; u < 8; ++u) out[i * N + (size_t)blk * 8 + u] = v[u] >= 0 ? (uint64_t)v[u] : q - (uint64_t)(-v[u]);
  }
}

void sample_small_rns(ckks_ctx* c, uint64_t* out, uint64_t seed, uint32_t kind, uint32_t a, uint32_t b, int dist,
                      int n_limbs, LimbMap map) {
  int nb = (c->N / 8 + SB - 1) / SB;
  hipLaunchKernelGGL(k_small, dim3(nb), dim3(SB), 0, c->stream, out, seed, kind, a, b, dist, n_limbs, map, c->log_n,
                     c->t.mods);
  HIPCHECK(hipGetLastError());
}

// b_i = e_i - a_i s_i + [i in digit] (P mod q_i) s'_i   (evaluation form)
__global__ void k_keyb(uint64_t* __restrict__ b, const uint64_t* __restrict__ a, const uint64_t* __restrict__ s,
                       const uint64_t* __restrict__ sp, int d_lo, int d_hi, const uint64_t* __restrict__ pmod,
                       int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const size_t j = blockIdx.x * (size_t)SB + threadIdx.x;
  const int i = blockIdx.y;
  const Mod m = mods[i];
  const size_t o = i * N + j;
  uint64_t v = sub_mod(b[o], reduce128((u128)a[o] * s[o], m), m.q);
  if (i >= d_lo && i < d_hi) v = add_mod(v, reduce128((u128)pmod[i] * sp[o], m), m.q);
  b[o] = v;
}

void keygen_swk(ckks_ctx* c, uint64_t seed, const uint64_t* s_ntt, const uint64_t* sp_ntt, uint64_t tag,
                uint64_t* key) {
  const size_t N = c->N;
  const int nm = c->n_mod();
  const LimbMap full = lm_q(nm);
  // P mod q_i for every Q prime
  std::vector<uint64_t> pm(nm, 0);
  for (int i = 0; i < c->L; ++i) {
    uint64_t v = 1;
    for (int k = 0; k < c->alpha; ++k) v = (uint64_t)((u128)v * (c->mod[c->L + k] % c->mod[i]) % c->mod[i]);
    pm[i] = v;
  }
  uint64_t* pmd = (uint64_t*)c->buf(10, nm * 8);
  HIPCHECK(hipMemcpyAsync(pmd, pm.data(), nm * 8, hipMemcpyHostToDevice, c->stream));
  for (int d = 0; d < c->beta(); ++d) {
    uint64_t* kb = key + ((size_t)d * 2 + 0) * nm * N;
    uint64_t* ka = key + ((size_t)d * 2 + 1) * nm * N;
    sample_uniform(c, ka, seed, 2, (uint32_t)tag, (uint32_t)d * 65536u, nm, full, 0);
    ntt_fwd(c, ka, nm, full, 1, 0);
    sample_small_rns(c, kb, seed, 3, (uint32_t)tag, (uint32_t)d, 1, nm, full);
    ntt_fwd(c, kb, nm, full, 1, 0);
    int lo = d * c->alpha, hi = std::min((d + 1) * c->alpha, c->L);
    hipLaunchKernelGGL(k_keyb, dim3(N / SB, nm), dim3(SB), 0, c->stream, kb, ka, s_ntt, sp_ntt, lo, hi, pmd,
                       c->log_n, c->t.mods);
    HIPCHECK(hipGetLastError());
  }
  // pm lives on the host stack: finish the upload before returning
  HIPCHECK(hipStreamSynchronize(c->stream));
}

// ---- sampling inside the transform --------------------------------------------------------------
// A forward transform begins with its column pass, and a tile of 8 or 16 columns takes as many consecutive
// coefficients of each row: whole blocks of the stream.  So the column pass draws its input instead of
// reading it (a small polynomial's blocks once for every limb), and of an encryption the row pass takes the
// rest: both polynomials' rows of a limb, then c0 = e - a s + m.
// Bound by the stream's 20 rounds (1060 instructions a block of 4 coefficients).  64 uniform polynomials of 7
// limbs at N = 2^16: 267 us, where drawing took 236 and the column pass 87.  One encryption of 7 limbs, bound by
// launch latency: 12.1 + 9.5 us in two kernels, 46 us in seven.
struct Draw {
  uint64_t seed;
  uint32_t kind, a;
  int32_t uniform;   // else CBD(21)
  int32_t pad;
};
// four coefficients as uniform4's, signed, for a prime of the fp64 range; r64 = 2^64 mod q.  A 64-bit half
// hi 2^32 + lo comes down as (hi 2^32 reduced) + lo, below 0.51 q.
__device__ __forceinline__ void uniform4_fp(const uint32_t (&w)[16], double r64, double qd, double qinv,
                                            uint64_t (&v)[4]) {
  auto half = [&](uint32_t hi, uint32_t lo) { return sred((double)hi * 4294967296.0, qd, qinv) + (double)lo; };
#pragma unroll
  for (int u = 0; u < 4; ++u)
    v[u] = f2b(sred(fmulmod_s(half(w[4 * u + 3], w[4 * u + 2]), r64, qd, qinv) + half(w[4 * u + 1], w[4 * u]), qd,
                    qinv));
}

// polynomial z's stream has the second nonce word d.a + z: the first one from d0, the others from d1
struct DrawSrc {
  Draw d0, d1;
  template <int LOGC, bool FP, int COLS>
  __device__ __forceinline__ void load(uint64_t (&x)[8], uint64_t* s, const MidPlace<LOGC, COLS>& p, int mi, const Mod& m,
                                       int z, const Tw& t, int log_n) const {
    typedef MidGeo<LOGC, COLS> G;
    const Draw d = z == 0 ? d0 : d1;
    const uint32_t first = blockIdx.x * COLS, nonce = d.a + (uint32_t)z;
    auto row = [&](int e) { return s + (e + (e >> 3)) * COLS; };
    uint32_t w[16];
    if (d.uniform) {
      const double r64 = FP ? fmulmod_s(4294967296.0, 4294967296.0, t.qd, t.qinv) : 0.0;
#pragma unroll 1
      for (int at = threadIdx.x; at < G::C * (COLS / 4); at += G::THREADS) {
        const int e = at / (COLS / 4), g = at % (COLS / 4) * 4;
        chacha_block(d.seed, d.kind, nonce, (uint32_t)mi, (((uint32_t)e << (log_n - LOGC)) + first + g) >> 2, w);
        uint64_t v[4];
        if (FP)
          uniform4_fp(w, r64, t.qd, t.qinv, v);
        else
          uniform4(w, m, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) row(e)[g + k] = v[k];
      }
    } else {
#pragma unroll 1
      for (int at = threadIdx.x; at < G::C * (COLS / 8); at += G::THREADS) {
        const int e = at / (COLS / 8), g = at % (COLS / 8) * 8;
        chacha_block(d.seed, d.kind, nonce, 0, (((uint32_t)e << (log_n - LOGC)) + first + g) >> 3, w);
        int64_t v[8];
        small8(w, 1, v);
#pragma unroll
        for (int k = 0; k < 8; ++k)
          row(e)[g + k] = FP ? f2b((double)(int32_t)v[k]) : v[k] >= 0 ? (uint64_t)v[k] : m.q - (uint64_t)(-v[k]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = s[p.a(u)];
  }
};

void expand_seeded(ckks_ctx* c, uint64_t a_seed, uint32_t ct_id0, size_t count, int level, uint64_t* cts) {
  const int l1 = level + 1;
  const size_t ct_words = 2 * (size_t)l1 * c->N;
  constexpr size_t CHUNK = 4096;   // polynomials per launch (grid z)
  for (size_t z0 = 0; z0 < count; z0 += CHUNK) {
    const size_t nz = std::min(CHUNK, count - z0);
    uint64_t* c1 = cts + z0 * ct_words + (size_t)l1 * c->N;
    const Draw d{a_seed, 4, ct_id0 + (uint32_t)z0, 1, 0};
    src_cols(c, c1, ct_words, DrawSrc{d, d}, l1, lm_q(l1), (int)nz);
    ntt_fwd_rows(c, c1, l1, lm_q(l1), (int)nz, ct_words);
  }
}

// One wave a polynomial (0: e and then c0, 1: a), both on the same chunks
template <int LOGC, bool FP>
__device__ __forceinline__ void enc_rows_body(uint64_t* l, uint64_t* c0, uint64_t* c1, const uint64_t* s,
                                              const uint64_t* m, const Mod& md, const Tw& t, int log_n) {
  constexpr int COLS = row_cols<LOGC>();
  typedef PassGeo<LOGC, COLS> G;
  constexpr int H = G::EPT / 2;
  const int poly = threadIdx.x >> 6;
  const Place<LOGC, COLS, true> p(threadIdx.x & 63, blockIdx.x);
  const uint64_t* in = poly ? c1 : c0;
  uint64_t* const mine = l + poly * G::LDS_WORDS;
  uint64_t x[G::EPT], sv[H], mv[H];
#pragma unroll
  for (int u = 0; u < G::EPT; ++u) x[u] = in[p.gidx(p.r + G::TPC * u, log_n)];
  // each wave takes half of the last step's elements
  auto elem = [&](int u) { return p.r + G::TPC * (u + poly * H); };
#pragma unroll
  for (int u = 0; u < H; ++u) {
    sv[u] = s[p.gidx(elem(u), log_n)];
    mv[u] = m[p.gidx(elem(u), log_n)];
  }
  fwd_core<LOGC, COLS, true, FP>(x, mine, p, t, log_n);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < G::EPT; ++u)
    mine[p.sidx(p.r * G::EPT + u)] = FP ? from_fbits(f2b(canon(b2f(x[u]), t.qd))) : canon8(x[u], t.c, t.q);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < H; ++u) {
    const uint32_t n = p.gidx(elem(u), log_n);
    const uint64_t e = l[p.sidx(elem(u))], a = l[G::LDS_WORDS + p.sidx(elem(u))];
    c1[n] = a;
    c0[n] = add_mod(sub_mod(e, mul_mod(a, sv[u], md), t.q), mv[u], t.q);
  }
}

template <int LOGC>
__global__ __launch_bounds__(128) void k_enc_rows(uint64_t* __restrict__ ct, int l1, const uint64_t* __restrict__ s,
                                                  const uint64_t* __restrict__ m, TwTables tt, int log_n) {
  __shared__ uint64_t l[2 * PassGeo<LOGC, row_cols<LOGC>()>::LDS_WORDS];
  const int i = blockIdx.y;
  const Mod md = cld(tt.mods + i);
  const size_t o = (size_t)i << log_n;
  uint64_t* c0 = ct + o;
  uint64_t* c1 = c0 + ((size_t)l1 << log_n);
  const Tw t = make_tw(tt.psi, tt.psi_s, tt.psi_f, md.q, md.qinv, i, log_n);
  if (fp_prime(md.q))
    enc_rows_body<LOGC, true>(l, c0, c1, s + o, m + o, md, t, log_n);
  else
    enc_rows_body<LOGC, false>(l, c0, c1, s + o, m + o, md, t, log_n);
}

void encrypt_sym(ckks_ctx* c, const uint64_t* s_ntt, const uint64_t* m_ntt, int level, uint64_t seed, uint64_t a_seed,
                 uint32_t ct_id, uint64_t* ct) {
  const int l1 = level + 1;
  src_cols(c, ct, (size_t)l1 * c->N, DrawSrc{Draw{seed, 5, ct_id, 0, 0}, Draw{a_seed, 4, ct_id - 1, 1, 0}}, l1,
           lm_q(l1), 2);
  const int lr = c->log_n - ntt_mid_log(c);
  const TwTables tt = tw_tables(c);
#define X(LC)                                                                                                       \
  hipLaunchKernelGGL(k_enc_rows<LC>, dim3((c->N >> LC) / row_cols<LC>(), l1), dim3(128), 0, c->stream, ct, l1, s_ntt, \
                     m_ntt, tt, c->log_n)
  switch (lr) {
    case 4: X(4); break;
    case 5: X(5); break;
    case 6: X(6); break;
    case 7: X(7); break;
    case 8: X(8); break;
    case 9: X(9); break;
    default: FICGCN_THROW(EINVAL_, "unsupported ring degree");
  }
#undef X
  HIPCHECK(hipGetLastError());
}

}  // namespace ficgcn
