// Canonical-embedding encoder and decoder on the device (server-side plaintexts: masks,
// weights; the client's inputs and results).  Slot j
// of m(X) is m(zeta^(5^j)), the N FFT inputs are the slot values at the odd
// powers of zeta (conjugates at zeta^(-5^j)), and
//   m_i = round_half_even( Re(exp(-i pi i / N) * FFT(v)_i) / N * scale ).
// The N-point FFT runs as two passes of N = N1 * N2 points (four-step form):
//   column pass: for each s2 < N2, the N1-point DFT over s1 of v[N2 s1 + s2],
//                times w^(s2 i1) (w = exp(-2 pi i / N)), back in place at N2 i1 + s2;
//   row pass   : for each i1 < N1, the N2-point DFT over s2 of that row, written
//                in natural order, FFT(v)_{i1 + N1 i2}.
// Each sub-DFT is an in-LDS radix-2 transform (bit-reversed load) of a block of
// COLS columns or rows.  The column pass gathers its input from the slot values, the
// row pass rounds and checks the 63-bit range, and the NTT's column pass takes every
// limb's residues from the rounded coefficients.  (24 plaintexts of 7 limbs at N = 2^16: 110 us
// on the device, with passes of their own to scatter, round and write residues 196 us.)
// Independent fp64 FFTs can round a coefficient differently when its scaled
// value sits within the FFT's error of a half-integer; decoding absorbs it.
//
// Decoding wants the N/2 values m(zeta^(5^j)) alone.  5^j = 4 t + 1, so with H = N/2
//   m(zeta^(4 t + 1)) = sum_{i < H} (m_i + i m_{i+H}) exp(i pi i / N) exp(2 pi i t i / H),
// an H-point transform of H complex inputs: conj FFT_H of (m_i - i m_{i+H}) exp(-i pi i / N), through the
// same two passes.  k_dec_lift makes those inputs from the residues.  Launch latency bounds a decryption (six
// small kernels, 61 us at N = 2^16 and 2 limbs); the exact lift and an N-point FFT on one host thread took
// 2.9 ms of 2.97 ms.  The root mean square error against extended precision is 0.89 to 0.94 times that
// transform's (N = 2^12 to 2^16).
#include "internal.h"
#include "ntt_dev.h"

namespace ficgcn {

typedef double2 cplx;

__device__ __forceinline__ cplx cmul(cplx a, cplx b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
// with fused multiply-adds (the decoder: one rounding fewer; the encoder's roundings stay as they are)
__device__ __forceinline__ cplx cmul_fma(cplx a, cplx b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return make_double2(a.x - b.x, a.y - b.y); }

constexpr int ET = 256;           // threads per block
constexpr int ENC_LDS = 32768;    // bytes of LDS per block: COLS * C complex values

// The transform's input and output.  Encoding: input g is the value of slot src[g] >> 1 (zero past n), its
// conjugate when src[g] is odd; output i gives the coefficient m_i, rounded half to even.
struct EncodeIo {
  const double *re, *im;
  size_t n;
  const uint32_t* src;
  const cplx* twist;
  double scale;
  int64_t* m;
  int* flag;
  __device__ __forceinline__ cplx in(const cplx*, size_t b, size_t g, int) const {
    const uint32_t u = src[g], j = u >> 1;
    const double x = j < n ? re[b * n + j] : 0.0;
    const double y = j < n && im ? im[b * n + j] : 0.0;
    return make_double2(x, u & 1 ? -y : y);
  }
  __device__ __forceinline__ void out(cplx*, size_t b, size_t i, int N, cplx x) const {
    const cplx t = twist[i];
    const double v = (t.x * x.x - t.y * x.y) / (double)N * scale;
    int64_t r = 0;
    if (fabs(v) < 9.2e18)
      r = (int64_t)rint(v);
    else
      *flag = 1;
    m[b * N + i] = r;
  }
};
// Decoding: complex values from and to memory
struct DecodeIo {
  cplx* V;
  __device__ __forceinline__ cplx in(const cplx* v, size_t b, size_t g, int N) const { return v[b * N + g]; }
  __device__ __forceinline__ void out(cplx*, size_t b, size_t i, int N, cplx x) const { V[b * N + i] = x; }
};

__device__ __forceinline__ uint32_t brev_bits(uint32_t x, int bits) { return __brev(x) >> (32 - bits); }

// w^e for e in [0, N): root holds w^k at RS k for k < N/2, and w^(k + N/2) = -w^k
template <int RS>
__device__ __forceinline__ cplx wpow(const cplx* __restrict__ root, uint32_t e, int N) {
  const uint32_t h = (uint32_t)N / 2;
  const cplx r = root[RS * (e < h ? e : e - h)];
  return e < h ? r : make_double2(-r.x, -r.y);
}

// One pass: COLS sub-DFTs of C points per block.  Column pass (ROW false):
// unit u = column s2, element s1 at N2 s1 + s2, result times w^(s2 i1) back in
// place.  Row pass: unit u = row i1, element s2 at N2 i1 + s2, result i2 to
// out[i1 + N1 i2].  RS: N is the ring degree (1, encoding) or its half (2, decoding), in the ring's table.
template <bool ROW, int RS, class Io>
__global__ __launch_bounds__(ET) void k_enc_fft(cplx* __restrict__ v, Io io, const cplx* __restrict__ root, int N, int N1, int N2, int logC,
                                                int COLS) {
  extern __shared__ cplx sh[];
  const int C = 1 << logC;
  const size_t b = blockIdx.y;
  const int u0 = blockIdx.x * COLS;
  cplx* vb = v + b * (size_t)N;
  const int total = COLS * C;
  // load, bit-reversed inside each unit; consecutive threads read consecutive words
  for (int t = threadIdx.x; t < total; t += ET) {
    int col, e;
    size_t g;
    if (ROW) {
      col = t / C;
      e = t % C;
      g = (size_t)N2 * (u0 + col) + e;
    } else {
      col = t % COLS;
      e = t / COLS;
      g = (size_t)N2 * e + u0 + col;
    }
    sh[col * C + brev_bits((uint32_t)e, logC)] = ROW ? vb[g] : io.in(v, b, g, N);
  }
  __syncthreads();
  // radix-2 stages, twiddles w_C^k = w^(k N / C)
  const int half_total = COLS * (C / 2);
  for (int len = 2; len <= C; len <<= 1) {
    const int half = len / 2;
    const int tstep = N / len;
    for (int t = threadIdx.x; t < half_total; t += ET) {
      const int col = t / (C / 2);
      const int bi = t % (C / 2);
      const int k = bi % half;
      const int i = (bi / half) * len + k;
      cplx* s = sh + col * C;
      const cplx w = root[RS * k * tstep];
      const cplx x0 = s[i], x1 = RS == 1 ? cmul(s[i + half], w) : cmul_fma(s[i + half], w);
      s[i] = cadd(x0, x1);
      s[i + half] = csub(x0, x1);
    }
    __syncthreads();
  }
  // store
  for (int t = threadIdx.x; t < total; t += ET) {
    if (ROW) {
      const int col = t % COLS, i2 = t / COLS;   // consecutive threads: consecutive rows i1
      io.out(v, b, (size_t)(u0 + col) + (size_t)N1 * i2, N, sh[col * C + i2]);
    } else {
      const int col = t % COLS, i1 = t / COLS;
      const uint32_t e = (uint32_t)(((uint64_t)(u0 + col) * (uint64_t)i1) % (uint64_t)N);
      const cplx w = wpow<RS>(root, e, N), y = sh[col * C + i1];
      vb[(size_t)N2 * i1 + u0 + col] = RS == 1 ? cmul(y, w) : cmul_fma(y, w);
    }
  }
}

// The transform's column pass reads the rounded coefficients, so the residues are never written in coefficient
// form: |r| < 2^63 as (its high half 2^32 reduced) + its low half, or Shoup's product with 1, in [0, 4q), and
// its negative
struct CoefSrc {
  const int64_t* m;
  const Fold25* folds;
  template <int LOGC, bool FP, int COLS>
  __device__ __forceinline__ void load(uint64_t (&x)[8], uint64_t*, const MidPlace<LOGC, COLS>& p, int mi, const Mod&, int z,
                                       const Tw& t, int log_n) const {
    const int64_t* a = m + ((size_t)z << log_n) + p.unit;
    const uint64_t one_s = FP ? 0 : cld(&folds[mi].one_s);
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = (uint64_t)a[(size_t)(p.r + MidGeo<LOGC>::TPC * u) << (log_n - LOGC)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t r = (int64_t)x[u];
      if (FP) {
        x[u] = f2b(sred((double)(int32_t)(r >> 32) * 4294967296.0, t.qd, t.qinv) + (double)(uint32_t)r);
      } else {
        const uint64_t v = mul_shoup_lazy4((uint64_t)(r < 0 ? -r : r), 1, one_s, t.c);
        x[u] = r < 0 ? t.c.q4 - v : v;
      }
    }
  }
};

static void ensure_enc_tables(ckks_ctx* c) {
  if (c->enc_root) return;
  std::vector<double> root, twist;
  std::vector<uint32_t> pos, src;
  encode_tables(c->N, root, twist, pos, src);
  HIPCHECK(hipMalloc(&c->enc_root, root.size() * 8));
  HIPCHECK(hipMemcpy(c->enc_root, root.data(), root.size() * 8, hipMemcpyHostToDevice));
  HIPCHECK(hipMalloc(&c->enc_twist, twist.size() * 8));
  HIPCHECK(hipMemcpy(c->enc_twist, twist.data(), twist.size() * 8, hipMemcpyHostToDevice));
  HIPCHECK(hipMalloc(&c->enc_pos, pos.size() * 4));
  HIPCHECK(hipMemcpy(c->enc_pos, pos.data(), pos.size() * 4, hipMemcpyHostToDevice));
  HIPCHECK(hipMalloc(&c->enc_src, src.size() * 4));
  HIPCHECK(hipMemcpy(c->enc_src, src.data(), src.size() * 4, hipMemcpyHostToDevice));
  HIPCHECK(hipMalloc(&c->enc_flag, sizeof(int)));
}

// the two passes over n_pt transforms of N points through v
template <int RS, class Io>
static void launch_fft(ckks_ctx* c, cplx* v, const Io& io, int n_pt, int N) {
  int l1 = 0;
  while ((1 << (2 * (l1 + 1))) <= N) ++l1;   // N1 = 2^floor(log N / 2)
  const int N1 = 1 << l1, N2 = N / N1;
  for (int row = 0; row < 2; ++row) {
    const int C = row ? N2 : N1, units = row ? N1 : N2;
    int logC = 0;
    while ((1 << logC) < C) ++logC;
    // a workgroup's LDS full of units, down to four (64-byte runs) where the grid would leave CUs idle
    int cols = std::min(ENC_LDS / (int)(C * sizeof(cplx)), units);
    while (cols > 4 && (int64_t)units / cols * n_pt < 256) cols /= 2;
    if (cols < 1 || units % cols) FICGCN_THROW(EINVAL_, "embedding FFT shape");
    hipLaunchKernelGGL(row ? (k_enc_fft<true, RS, Io>) : (k_enc_fft<false, RS, Io>), dim3(units / cols, n_pt), dim3(ET),
                       (size_t)cols * C * sizeof(cplx), c->stream, v, io, (const cplx*)c->enc_root, N, N1, N2, logC,
                       cols);
    HIPCHECK(hipGetLastError());
  }
}

void encode_gpu(ckks_ctx* c, const double* re, const double* im, size_t count, size_t n, double scale, int n_limbs,
                LimbMap map, uint64_t* dev) {
  if (count == 0) return;
  if (n > (size_t)c->N / 2) FICGCN_THROW(EINVAL_, "more values than slots");
  if (!re && n > 0) FICGCN_THROW(EINVAL_, "null slot values");
  ensure_enc_tables(c);
  const int N = c->N;
  // chunks of plaintexts: slot values, the FFT buffer and the coefficients
  const size_t CH = 32;
  const size_t nn = n > 0 ? n : 1;
  double* d_re = (double*)dev_scratch(c, 17, CH * nn * 8 * (im ? 2 : 1));
  double* d_im = im ? d_re + CH * nn : nullptr;
  cplx* v = (cplx*)dev_scratch(c, 18, CH * (size_t)N * sizeof(cplx));
  int64_t* m = (int64_t*)dev_scratch(c, 19, CH * (size_t)N * 8);
  HIPCHECK(hipMemsetAsync(c->enc_flag, 0, sizeof(int), c->stream));
  for (size_t b0 = 0; b0 < count; b0 += CH) {
    const int nb = (int)std::min(CH, count - b0);
    if (n > 0) {
      HIPCHECK(hipMemcpyAsync(d_re, re + b0 * n, (size_t)nb * n * 8, hipMemcpyHostToDevice, c->stream));
      if (im) HIPCHECK(hipMemcpyAsync(d_im, im + b0 * n, (size_t)nb * n * 8, hipMemcpyHostToDevice, c->stream));
    }
    launch_fft<1>(c, v, EncodeIo{d_re, d_im, n, c->enc_src, (const cplx*)c->enc_twist, scale, m, c->enc_flag}, nb, N);
    uint64_t* pt = dev + b0 * (size_t)n_limbs * N;
    const size_t stride = (size_t)n_limbs * N;
    src_cols(c, pt, stride, CoefSrc{m, c->t.fold25}, n_limbs, map, nb);
    ntt_fwd_rows(c, pt, n_limbs, map, nb, stride);
    // the host slot values of this chunk are re-read by the next chunk's copy only after this point
    HIPCHECK(hipStreamSynchronize(c->stream));
  }
  int flag = 0;
  HIPCHECK(hipMemcpy(&flag, c->enc_flag, sizeof(int), hipMemcpyDeviceToHost));
  if (flag) FICGCN_THROW(ESCALE_, "encoded coefficient exceeds 63 bits");
}

// The centred value of k residues, divided by scale.  Mixed radix digits, x = v_0 + q_0 (v_1 + q_1 (v_2 + ..)):
//   v_i = (..((r_i - v_0) / q_0 - v_1) / q_1 ..) / q_{i-1} mod q_i,
// written over the residues.  Every q is odd, so (Q - 1) / 2 has the digits (q_i - 1) / 2 and Q - 1 - x the
// digits q_i - 1 - v_i: comparing and negating go digit by digit.  The digits are summed from the top in
// pairs of doubles: two of 50 bits (and all below 2^106) come out rounded once, more of them within that
// rounding and 2^-100.
__device__ double lift(uint64_t* __restrict__ m, size_t N, int k, double scale, const uint64_t* __restrict__ inv,
                       int L, const Mod* __restrict__ mods) {
  struct W2 {
    uint64_t w, s;
  };
  const W2* iv = (const W2*)inv;
  for (int i = 1; i < k; ++i) {
    const uint64_t q = cld(&mods[i].q);
    uint64_t t = m[i * N];
    for (int j = 0; j < i; ++j) {
      const W2 u = cld(iv + (size_t)i * L + j);
      t = sub_mod(mul_shoup(t, u.w, u.s, q), mul_shoup(m[j * N], u.w, u.s, q), q);
    }
    m[i * N] = t;
  }
  bool neg = false;
  for (int i = k - 1; i >= 0; --i) {
    const uint64_t half = (cld(&mods[i].q) - 1) >> 1, v = m[i * N];
    if (v != half) {
      neg = v > half;
      break;
    }
  }
  double hi = 0, lo = 0;
  auto add = [&](uint64_t v) {
    const double x = (double)v, xl = (double)(int64_t)(v - (uint64_t)x);
    const double s = hi + x, b = s - hi;
    const double e = ((hi - (s - b)) + (x - b)) + (lo + xl);
    hi = s + e;
    lo = e - (hi - s);
  };
  for (int i = k - 1; i >= 0; --i) {
    const uint64_t q = cld(&mods[i].q), v = m[i * N];
    const double x = (double)q, xl = (double)(int64_t)(q - (uint64_t)x);
    const double p = hi * x;
    const double e = fma(hi, x, -p) + (hi * xl + lo * x);
    hi = p + e;
    lo = e - (hi - p);
    add(neg ? q - 1 - v : v);
  }
  if (neg) add(1);
  return (neg ? -hi : hi) / scale;
}

// v_i = (m_i - i m_{i+H}) exp(-i pi i / N), two threads an i (k^2 / 2 modular products a coefficient)
__global__ __launch_bounds__(ET) void k_dec_lift(uint64_t* __restrict__ m, int N, int k, double scale,
                                                 const uint64_t* __restrict__ inv, int L,
                                                 const Mod* __restrict__ mods, const cplx* __restrict__ twist,
                                                 cplx* __restrict__ v) {
  __shared__ double x[ET];
  const int h = threadIdx.x / (ET / 2), u = threadIdx.x % (ET / 2);
  const size_t i = blockIdx.x * (size_t)(ET / 2) + u;
  const size_t at = i + (size_t)h * (N / 2);
  x[threadIdx.x] = i < (size_t)N / 2 ? lift(m + at, N, k, scale, inv, L, mods) : 0.0;
  __syncthreads();
  if (h == 0 && i < (size_t)N / 2) v[i] = cmul_fma(make_double2(x[u], -x[u + ET / 2]), twist[i]);
}

// slot j is the conjugate of V_t, t = pos[j], 4 t + 1 = 5^j.  The results go straight to host memory.
__global__ void k_dec_gather(const cplx* __restrict__ V, const uint32_t* __restrict__ pos, size_t n,
                             double* __restrict__ re, double* __restrict__ im) {
  const size_t j = blockIdx.x * (size_t)ET + threadIdx.x;
  if (j >= n) return;
  const cplx x = V[pos[j]];
  re[j] = x.x;
  im[j] = -x.y;
}

static void ensure_dec_tables(ckks_ctx* c) {
  ensure_enc_tables(c);
  if (!c->dec_inv) {
    std::vector<uint64_t> t((size_t)c->L * c->L * 2, 0);
    for (int i = 0; i < c->L; ++i)
      for (int j = 0; j < i; ++j) {
        const uint64_t q = c->mod[i], w = invmod(c->mod[j] % q, q);
        t[((size_t)i * c->L + j) * 2] = w;
        t[((size_t)i * c->L + j) * 2 + 1] = shoup(w, q);
      }
    HIPCHECK(hipMalloc(&c->dec_inv, t.size() * 8));
    HIPCHECK(hipMemcpy(c->dec_inv, t.data(), t.size() * 8, hipMemcpyHostToDevice));
  }
  if (!c->dec_host) HIPCHECK(hipHostMalloc(&c->dec_host, (size_t)c->N * 8, hipHostMallocDefault));
}

void decode_gpu(ckks_ctx* c, uint64_t* m, int k, double scale, double* re, double* im, size_t n) {
  ensure_dec_tables(c);
  const size_t N = c->N, H = N / 2;
  if (n > H) FICGCN_THROW(EINVAL_, "more values than slots");
  if (n > 0) {
    cplx* v = (cplx*)dev_scratch(c, 18, H * sizeof(cplx));
    cplx* V = (cplx*)dev_scratch(c, 19, H * sizeof(cplx));
    hipLaunchKernelGGL(k_dec_lift, dim3((H + ET / 2 - 1) / (ET / 2)), dim3(ET), 0, c->stream, m, (int)N, k, scale,
                       c->dec_inv, c->L, c->t.mods, (const cplx*)c->enc_twist, v);
    HIPCHECK(hipGetLastError());
    launch_fft<2>(c, v, DecodeIo{V}, 1, (int)H);
    hipLaunchKernelGGL(k_dec_gather, dim3((n + ET - 1) / ET), dim3(ET), 0, c->stream, V, c->enc_pos, n, c->dec_host,
                       c->dec_host + H);
    HIPCHECK(hipGetLastError());
  }
  HIPCHECK(hipStreamSynchronize(c->stream));
  if (re) std::copy_n(c->dec_host, n, re);
  if (im) std::copy_n(c->dec_host + H, n, im);
}

}  // namespace ficgcn
