// CKKS context: prime chain, NTT twiddle tables, base-conversion constants.
//
// Prime chain (paper Sec. 2.1: Q = q_0 ... q_{L-1}): the L largest primes
// below 2^q_bits with q = 1 (mod 2N), in descending order, then the alpha
// largest primes below 2^p_bits with p = 1 (mod 2N) as the special modulus P
// of hybrid key switching.
#include <algorithm>
#include <cstring>
#include <stdexcept>
#include <thread>

#include "internal.h"

namespace ficgcn {

uint64_t powmod(uint64_t a, uint64_t e, uint64_t q) {
  uint64_t r = 1 % q;
  a %= q;
  while (e) {
    if (e & 1) r = (uint64_t)((u128)r * a % q);
    a = (uint64_t)((u128)a * a % q);
    e >>= 1;
  }
  return r;
}

uint64_t invmod(uint64_t a, uint64_t q) { return powmod(a, q - 2, q); }

uint64_t shoup(uint64_t w, uint64_t q) { return (uint64_t)(((u128)w << 64) / q); }

Mod make_mod(uint64_t q) {
  // floor(2^128 / q) = floor((2^128 - 1) / q) for q not a power of two
  u128 all = ~(u128)0;
  u128 r = all / q;
  return Mod{q, (uint64_t)(r >> 64), (uint64_t)r, 1.0 / (double)q};
}

static bool miller_rabin(uint64_t n) {
  if (n < 2) return false;
  static const uint64_t bases[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
  for (uint64_t p : bases)
    if (n % p == 0) return n == p;
  uint64_t d = n - 1;
  int s = 0;
  while ((d & 1) == 0) { d >>= 1; ++s; }
  for (uint64_t a : bases) {
    uint64_t x = powmod(a, d, n);
    if (x == 1 || x == n - 1) continue;
    bool comp = true;
    for (int r = 1; r < s; ++r) {
      x = (uint64_t)((u128)x * x % n);
      if (x == n - 1) { comp = false; break; }
    }
    if (comp) return false;
  }
  return true;
}

static std::vector<uint64_t> chain(int bits, int count, uint64_t two_n, const std::vector<uint64_t>& avoid) {
  std::vector<uint64_t> out;
  uint64_t top = (bits >= 64) ? ~0ull : ((1ull << bits) - 1);
  uint64_t p = top / two_n * two_n + 1;
  if (p > top) p -= two_n;
  while ((int)out.size() < count) {
    if (p < two_n) FICGCN_THROW(EINVAL_, "not enough NTT primes of this size");
    bool skip = false;
    for (uint64_t a : avoid) skip |= (a == p);
    if (!skip && miller_rabin(p)) out.push_back(p);
    p -= two_n;
  }
  return out;
}

static uint64_t root_2n(uint64_t q, uint64_t two_n) {
  uint64_t e = (q - 1) / two_n;
  for (uint64_t x = 2;; ++x) {
    uint64_t psi = powmod(x, e, q);
    if (powmod(psi, two_n / 2, q) == q - 1) return psi;
  }
}

static uint32_t brev_host(uint32_t x, int bits) {
  uint32_t r = 0;
  for (int i = 0; i < bits; ++i) r |= ((x >> i) & 1u) << (bits - 1 - i);
  return r;
}

void build_context(ckks_ctx* c) {
  c->N = 1 << c->log_n;
  uint64_t two_n = 2ull * c->N;
  if (c->q_bits > 61 || c->p_bits > 61 || c->q_bits < 20 || c->p_bits < 20)
    FICGCN_THROW(EINVAL_, "prime sizes must be in [20, 61] bits");
  std::vector<uint64_t> q = chain(c->q_bits, c->L, two_n, {});
  std::vector<uint64_t> p = chain(c->p_bits, c->alpha, two_n, q);
  c->mod = q;
  c->mod.insert(c->mod.end(), p.begin(), p.end());
  int nm = c->n_mod();
  size_t N = c->N;
  std::vector<uint64_t> psi(nm * N), psi_s(nm * N), ipsi(nm * N), ipsi_s(nm * N), ninv(nm), ninv_s(nm);
  std::vector<Mod> mods(nm);
  c->psi.resize(nm);
  std::vector<std::thread> th;
  for (int m = 0; m < nm; ++m) {
    th.emplace_back([&, m]() {
      uint64_t qm = c->mod[m];
      uint64_t r = root_2n(qm, two_n);
      c->psi[m] = r;
      uint64_t ir = invmod(r, qm);
      // powers in natural order, then placed at bit-reversed positions
      std::vector<uint64_t> pw(N), ipw(N);
      pw[0] = 1;
      ipw[0] = 1;
      for (size_t k = 1; k < N; ++k) {
        pw[k] = (uint64_t)((u128)pw[k - 1] * r % qm);
        ipw[k] = (uint64_t)((u128)ipw[k - 1] * ir % qm);
      }
      for (size_t k = 0; k < N; ++k) {
        uint32_t b = brev_host((uint32_t)k, c->log_n);
        psi[m * N + k] = pw[b];
        psi_s[m * N + k] = shoup(pw[b], qm);
        ipsi[m * N + k] = ipw[b];
        ipsi_s[m * N + k] = shoup(ipw[b], qm);
      }
      ninv[m] = invmod(N % qm, qm);
      ninv_s[m] = shoup(ninv[m], qm);
      mods[m] = make_mod(qm);
    });
  }
  for (auto& t : th) t.join();
  c->h_psi.swap(psi);
  c->h_psi_s.swap(psi_s);
  c->h_ipsi.swap(ipsi);
  c->h_ipsi_s.swap(ipsi_s);
  c->h_ninv.swap(ninv);
  c->h_ninv_s.swap(ninv_s);
  c->h_mods.swap(mods);
}

// ModDown and rescale constants of every level.  h = floor(P / 2) = (P - 1) / 2 (P odd), so its
// residue modulo m is (P mod m - 1) 2^-1 mod m.
static void level_constants(ckks_ctx* c) {
  auto p_mod = [&](uint64_t m) {
    uint64_t v = 1;
    for (int u = 0; u < c->alpha; ++u) v = (uint64_t)((u128)v * (c->mod[c->L + u] % m) % m);
    return v;
  };
  MDK all{};
  for (int t = 0; t < c->alpha; ++t) {
    const uint64_t pm = c->mod[c->L + t];
    all.hP[t] = (uint64_t)((u128)sub_mod(p_mod(pm), 1, pm) * invmod(2, pm) % pm);
  }
  c->mdk.assign(c->L, MDK{});
  c->rsk.assign(c->L, RSK{});
  for (int level = 0; level < c->L; ++level) {
    const uint64_t q = c->mod[level], P = p_mod(q);
    all.hQ[level] = (uint64_t)((u128)sub_mod(P, 1, q) * invmod(2, q) % q);
    all.pinv[level] = invmod(P, q);
    all.pinv_s[level] = shoup(all.pinv[level], q);
    c->mdk[level] = all;
    RSK& r = c->rsk[level];
    for (int i = 0; i < level; ++i) {
      const uint64_t qi = c->mod[i];
      r.h[i] = (q / 2) % qi;
      r.inv[i] = invmod(q % qi, qi);
      r.inv_s[i] = shoup(r.inv[i], qi);
    }
  }
}

// The maps of the transforms fused with base conversions (ntt_fused.hip), for every level:
// one table of source and destination entries for ModUp's digits, ModDown and the two rescales.
static void mid_tables(ckks_ctx* c) {
  std::vector<MidSrc> src;
  std::vector<MidDst> dst;
  auto source = [&](int mi, uint64_t scale, uint64_t shift) {
    const uint64_t q = c->mod[mi];
    MidSrc s{};
    s.q = q;
    s.qinv = 1.0 / (double)q;
    s.c = scale;
    s.cs = shoup(scale, q);
    s.sh = shift;
    s.mi = mi;
    return s;
  };
  auto dest = [&](int mi, int pos) {
    MidDst d{};
    d.q = c->mod[mi];
    d.qinv = 1.0 / (double)d.q;
    d.mi = mi;
    d.pos = pos;
    return d;
  };
  // product of the other sources' primes modulo m
  auto hat = [&](const std::vector<int>& srcs, int t, uint64_t m) {
    uint64_t v = 1;
    for (int u = 0; u < (int)srcs.size(); ++u)
      if (u != t) v = (uint64_t)((u128)v * (c->mod[srcs[u]] % m) % m);
    return v;
  };
  auto mul = [](uint64_t a, uint64_t b, uint64_t q) { return (uint64_t)((u128)a * b % q); };
  // fast base conversion of `srcs` (at most two) to the listed destinations; half: ModDown's rounding
  auto bconv = [&](const std::vector<int>& srcs, const std::vector<std::pair<int, int>>& dsts, const MDK* half) {
    for (int t = 0; t < 2; ++t) {
      if (t >= (int)srcs.size()) {
        src.push_back(MidSrc{});
        continue;
      }
      const uint64_t q = c->mod[srcs[t]], inv = invmod(hat(srcs, t, q), q);
      src.push_back(source(srcs[t], mul(inv, c->h_ninv[srcs[t]], q), half ? mul(half->hP[t], inv, q) : 0));
    }
    for (const auto& d : dsts) {
      MidDst e = dest(d.first, d.second);
      for (int t = 0; t < (int)srcs.size(); ++t) {
        e.a[t] = hat(srcs, t, e.q);
        e.a[2 + t] = shoup(e.a[t], e.q);
      }
      e.a[4] = half ? half->hQ[d.second] : 0;
      dst.push_back(e);
    }
  };
  const int a = c->alpha;
  c->mid.assign(c->L, MidLevel{});
  for (int level = 0; level < c->L; ++level) {
    MidLevel& m = c->mid[level];
    const int l1 = level + 1, ext = l1 + a;
    if (a <= 2) {
      m.up_s = src.size();
      m.up_d = dst.size();
      for (int d = 0; d * a < l1; ++d) {
        const int lo = d * a, hi = std::min(lo + a, l1);
        std::vector<int> s;
        std::vector<std::pair<int, int>> to;
        for (int i = lo; i < hi; ++i) s.push_back(i);
        for (int i = 0; i < l1; ++i)
          if (i < lo || i >= hi) to.push_back({i, i});
        for (int k = 0; k < a; ++k) to.push_back({c->L + k, l1 + k});
        bconv(s, to, nullptr);
        while ((int)(dst.size() - m.up_d) < (d + 1) * ext) dst.push_back(MidDst{});   // ext entries a digit
      }
      m.down_s = src.size();
      m.down_d = dst.size();
      std::vector<int> s;
      std::vector<std::pair<int, int>> to;
      for (int k = 0; k < a; ++k) s.push_back(c->L + k);
      for (int i = 0; i < l1; ++i) to.push_back({i, i});
      bconv(s, to, &c->mdk[level]);
    }
    if (level >= 1) {
      const RSK& r = c->rsk[level];
      const uint64_t ql = c->mod[level];
      m.rs_s = src.size();
      m.rs_d = dst.size();
      src.push_back(source(level, c->h_ninv[level], ql / 2));
      for (int i = 0; i < level; ++i) {
        MidDst e = dest(i, i);
        e.a[0] = r.h[i];
        dst.push_back(e);
      }
    }
    if (level >= 2) {
      const RSK &r1 = c->rsk[level], &r2 = c->rsk[level - 1];
      m.rs2_s = src.size();
      m.rs2_d = dst.size();
      // limb l-1 gets its half after the first correction (e), limb l its own at once
      MidSrc lower = source(level - 1, c->h_ninv[level - 1], 0);
      lower.e[0] = r1.h[level - 1];
      lower.e[1] = r1.inv[level - 1];
      lower.e[2] = r1.inv_s[level - 1];
      src.push_back(lower);
      src.push_back(source(level, c->h_ninv[level], c->mod[level] / 2));
      for (int i = 0; i < level - 1; ++i) {
        MidDst e = dest(i, i);
        const uint64_t v[6] = {r1.h[i], r2.h[i], r1.inv[i], r1.inv_s[i], r2.inv[i], r2.inv_s[i]};
        std::copy(v, v + 6, e.a);
        dst.push_back(e);
      }
    }
  }
  HIPCHECK(hipMalloc(&c->mid_src, std::max<size_t>(1, src.size()) * sizeof(MidSrc)));
  HIPCHECK(hipMemcpy(c->mid_src, src.data(), src.size() * sizeof(MidSrc), hipMemcpyHostToDevice));
  HIPCHECK(hipMalloc(&c->mid_dst, std::max<size_t>(1, dst.size()) * sizeof(MidDst)));
  HIPCHECK(hipMemcpy(c->mid_dst, dst.data(), dst.size() * sizeof(MidDst), hipMemcpyHostToDevice));
}

void ensure_device(ckks_ctx* c) {
  if (c->on_device) return;
  HIPCHECK(hipGetDevice(&c->device));
  auto up = [&](uint64_t** dst, const std::vector<uint64_t>& v) {
    HIPCHECK(hipMalloc(dst, v.size() * 8));
    HIPCHECK(hipMemcpy(*dst, v.data(), v.size() * 8, hipMemcpyHostToDevice));
  };
  up(&c->t.psi, c->h_psi);
  up(&c->t.psi_s, c->h_psi_s);
  up(&c->t.ipsi, c->h_ipsi);
  up(&c->t.ipsi_s, c->h_ipsi_s);
  auto up_f = [&](double** dst, const std::vector<uint64_t>& v) {
    std::vector<double> f(v.size());
    for (size_t i = 0; i < v.size(); ++i) f[i] = (double)v[i];
    HIPCHECK(hipMalloc(dst, f.size() * 8));
    HIPCHECK(hipMemcpy(*dst, f.data(), f.size() * 8, hipMemcpyHostToDevice));
  };
  up_f(&c->t.psi_f, c->h_psi);
  up_f(&c->t.ipsi_f, c->h_ipsi);
  up(&c->t.ninv, c->h_ninv);
  up(&c->t.ninv_s, c->h_ninv_s);
  HIPCHECK(hipMalloc(&c->t.mods, c->h_mods.size() * sizeof(Mod)));
  HIPCHECK(hipMemcpy(c->t.mods, c->h_mods.data(), c->h_mods.size() * sizeof(Mod), hipMemcpyHostToDevice));
  std::vector<Fold25> fold(c->n_mod());
  for (int m = 0; m < c->n_mod(); ++m) {
    const uint64_t q = c->mod[m], r25 = (1ull << 25) % q, r50 = (1ull << 50) % q;
    uint64_t P = 1;
    for (int k = 0; k < c->alpha; ++k) P = (uint64_t)((u128)P * (c->mod[c->L + k] % q) % q);
    fold[m] = Fold25{r25, shoup(r25, q), r50, shoup(r50, q), shoup(1, q), P};
  }
  HIPCHECK(hipMalloc(&c->t.fold25, fold.size() * sizeof(Fold25)));
  HIPCHECK(hipMemcpy(c->t.fold25, fold.data(), fold.size() * sizeof(Fold25), hipMemcpyHostToDevice));
  // every base-conversion table of the chain, so later calls find them built
  for (int level = 0; level < c->L; ++level) {
    for (int d = 0; d * c->alpha <= level; ++d) get_modup(c, level, d);
    get_moddown(c, level);
  }
  level_constants(c);
  mid_tables(c);
  c->on_device = true;
}

// FastBConv constants: hat_b = prod_{s' != s} b_{s'}; hat_inv[s] = hat_b^-1 mod b_s;
// hat_mod[d][s] = hat_b mod p_d.
static BConv make_bconv(ckks_ctx* c, const std::vector<int>& src, const std::vector<int>& dst) {
  BConv bc;
  bc.src = src;
  bc.dst = dst;
  bc.n_src = (int)src.size();
  bc.n_dst = (int)dst.size();
  std::vector<uint64_t> h(2 * bc.n_src + bc.n_dst * bc.n_src);
  for (int s = 0; s < bc.n_src; ++s) {
    uint64_t bs = c->mod[src[s]];
    uint64_t hat = 1;
    for (int s2 = 0; s2 < bc.n_src; ++s2)
      if (s2 != s) hat = (uint64_t)((u128)hat * (c->mod[src[s2]] % bs) % bs);
    h[s] = invmod(hat, bs);
    h[bc.n_src + s] = shoup(h[s], bs);
  }
  for (int d = 0; d < bc.n_dst; ++d) {
    uint64_t pd = c->mod[dst[d]];
    for (int s = 0; s < bc.n_src; ++s) {
      uint64_t hat = 1;
      for (int s2 = 0; s2 < bc.n_src; ++s2)
        if (s2 != s) hat = (uint64_t)((u128)hat * (c->mod[src[s2]] % pd) % pd);
      h[2 * bc.n_src + d * bc.n_src + s] = hat;
    }
  }
  HIPCHECK(hipMalloc(&bc.dev, h.size() * 8));
  HIPCHECK(hipMemcpy(bc.dev, h.data(), h.size() * 8, hipMemcpyHostToDevice));
  std::vector<int> ix(src);
  ix.insert(ix.end(), dst.begin(), dst.end());
  HIPCHECK(hipMalloc(&bc.idx, ix.size() * sizeof(int)));
  HIPCHECK(hipMemcpy(bc.idx, ix.data(), ix.size() * sizeof(int), hipMemcpyHostToDevice));
  return bc;
}

// ModUp of digit `digit` at `level`: source = the digit's active Q primes,
// destinations = every other active Q prime, then the P primes.
const BConv& get_modup(ckks_ctx* c, int level, int digit) {
  auto key = std::make_pair(level, digit);
  auto it = c->modup.find(key);
  if (it != c->modup.end()) return it->second;
  std::vector<int> src, dst;
  int lo = digit * c->alpha, hi = std::min((digit + 1) * c->alpha, level + 1);
  for (int i = lo; i < hi; ++i) src.push_back(i);
  for (int i = 0; i <= level; ++i)
    if (i < lo || i >= hi) dst.push_back(i);
  for (int k = 0; k < c->alpha; ++k) dst.push_back(c->L + k);
  return c->modup[key] = make_bconv(c, src, dst);
}

const BConv& get_moddown(ckks_ctx* c, int level) {
  auto it = c->moddown.find(level);
  if (it != c->moddown.end()) return it->second;
  std::vector<int> src, dst;
  for (int k = 0; k < c->alpha; ++k) src.push_back(c->L + k);
  for (int i = 0; i <= level; ++i) dst.push_back(i);
  return c->moddown[level] = make_bconv(c, src, dst);
}

uint64_t galois_elt(ckks_ctx* c, int64_t step) {
  int64_t M = c->N / 2;
  int64_t k = ((step % M) + M) % M;
  return powmod(5, (uint64_t)k, 2ull * c->N);
}

}  // namespace ficgcn

namespace ficgcn {

Recorder::~Recorder() {
  for (auto& b : bufs)
    if (b.first) (void)hipFree(b.first);
}

static void* recorded(ckks_ctx* c, size_t bytes, const void* host) {
  Recorder* r = c->rec;
  if (r->mode == Recorder::RECORD) {
    void* d = nullptr;
    HIPCHECK(hipMalloc(&d, std::max<size_t>(16, bytes)));
    r->bufs.push_back({d, bytes});
    if (host && bytes) {
      HIPCHECK(hipStreamSynchronize(c->stream));
      HIPCHECK(hipMemcpy(d, host, bytes, hipMemcpyHostToDevice));
    }
    return d;
  }
  if (r->cursor >= r->bufs.size() || r->bufs[r->cursor].second != bytes)
    FICGCN_THROW(EPLAN_, "replayed launch sequence differs from the recorded one");
  return r->bufs[r->cursor++].first;
}

void* dev_scratch(ckks_ctx* c, int slot, size_t bytes) {
  if (c->rec) return recorded(c, bytes, nullptr);
  return c->buf(slot, bytes);
}

// Small tables go through a ring of pinned memory and its device twin: a kernel copies each into place in stream
// order, so the caller's list may go and no launch waits for the host.  A table keeps its words while the ring's
// next lap is at least STAGE_RING - 2 STAGE_MAX bytes away; a lap begins after a wait for the stream.  Larger ones
// are copied from pageable memory, and waited for.  A small network of 128 launches took 955 us with a copy from
// pageable memory for each of its 34 tables and a wait after each of its batches, 729 us this way.
constexpr size_t STAGE_RING = 2 << 20, STAGE_MAX = 256 << 10;
void* dev_table(ckks_ctx* c, int slot, const void* host, size_t bytes) {
  if (c->rec) return recorded(c, bytes, host);
  if (bytes > STAGE_MAX) {
    void* d = c->buf(slot, bytes);
    HIPCHECK(hipMemcpyAsync(d, host, bytes, hipMemcpyHostToDevice, c->stream));
    HIPCHECK(hipStreamSynchronize(c->stream));
    return d;
  }
  if (!c->stage_host) HIPCHECK(hipHostMalloc(&c->stage_host, STAGE_RING, hipHostMallocDefault));
  if (!c->stage_dev) HIPCHECK(hipMalloc(&c->stage_dev, STAGE_RING));
  const size_t room = std::max<size_t>(16, (bytes + 15) & ~(size_t)15);
  if (c->stage_at + room > STAGE_RING) {
    HIPCHECK(hipStreamSynchronize(c->stream));
    c->stage_at = 0;
  }
  const size_t at = c->stage_at;
  c->stage_at += room;
  if (bytes) {
    std::memcpy(c->stage_host + at, host, bytes);
    stage_copy(c, c->stage_dev + at, c->stage_host + at, room);
  }
  return c->stage_dev + at;
}

void stream_sync(ckks_ctx* c) {
  if (c->rec && c->rec->mode == Recorder::REPLAY) return;
  HIPCHECK(hipStreamSynchronize(c->stream));
}

}  // namespace ficgcn

void* ckks_ctx::buf(int slot, size_t bytes) {
  if ((int)scratch.size() <= slot) scratch.resize(slot + 1, {nullptr, 0});
  auto& s = scratch[slot];
  if (s.second < bytes) {
    if (s.first) {
      HIPCHECK(hipStreamSynchronize(stream));
      HIPCHECK(hipFree(s.first));
    }
    s.first = nullptr;
    HIPCHECK(hipMalloc(&s.first, bytes));
    s.second = bytes;
  }
  return s.first;
}

ckks_ctx::~ckks_ctx() {
  if (stream) (void)hipStreamSynchronize(stream);
  for (auto& s : scratch)
    if (s.first) (void)hipFree(s.first);
  for (uint64_t* p : {t.psi, t.psi_s, t.ipsi, t.ipsi_s, t.ninv, t.ninv_s})
    if (p) (void)hipFree(p);
  for (double* p : {t.psi_f, t.ipsi_f, enc_root, enc_twist})
    if (p) (void)hipFree(p);
  if (enc_pos) (void)hipFree(enc_pos);
  if (enc_src) (void)hipFree(enc_src);
  if (enc_flag) (void)hipFree(enc_flag);
  if (dec_inv) (void)hipFree(dec_inv);
  if (dec_host) (void)hipHostFree(dec_host);
  if (stage_host) (void)hipHostFree(stage_host);
  if (stage_dev) (void)hipFree(stage_dev);
  if (t.mods) (void)hipFree(t.mods);
  if (t.fold25) (void)hipFree(t.fold25);
  if (mid_src) (void)hipFree(mid_src);
  if (mid_dst) (void)hipFree(mid_dst);
  for (auto& kv : modup) { (void)hipFree(kv.second.dev); (void)hipFree(kv.second.idx); }
  for (auto& kv : moddown) { (void)hipFree(kv.second.dev); (void)hipFree(kv.second.idx); }
}

ckks_keys::~ckks_keys() {
  if (ctx && ctx->stream) (void)hipStreamSynchronize(ctx->stream);
  if (s_ntt) (void)hipFree(s_ntt);
  for (auto& kv : swk) (void)hipFree(kv.second);
}
