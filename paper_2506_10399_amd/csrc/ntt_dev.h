// The NTT's butterflies and in-register sub-transforms (device code), shared by the plain passes
// (ntt.hip), the passes fused with base conversion (ntt_fused.hip) and those that make their own input
// (sample.hip, encode_gpu.hip).
#pragma once
#include <type_traits>

#include "fpmod.h"
#include "internal.h"
#include "ks_common.h"

namespace ficgcn {

// Integer butterflies with lazy reduction (after Harvey, for q < 2^61): inside a forward transform
// the values lie in [0, 8q), inside an inverse one in [0, 4q).
//
// Shoup's product a w mod q for any 64-bit a, with the quotient's estimate cut short: of
// a ws = a1 s1 2^64 + (a0 s1 + a1 s0) 2^32 + a0 s0 (32-bit halves) only a1 s1 and the high words of
// the two middle products are kept.  That loses less than 3 of the exact a w / q - a / 2^64, so
// r = a w - h q lies in [0, 4q): thirteen instructions, where the exact high product takes twenty.
// The 64-bit additions below go through v_lshl_add_u64: negated constants are kept opaque and
// differences are sums with a complement, since a borrow chain (v_sub_co, v_subb_co) and a compare
// with its selects take more instructions and wait states between them.
struct IntQ {
  uint64_t nq;     // -q
  uint64_t q4;     // 4q
  uint64_t nq4;    // -4q
  uint64_t q4p1;   // 4q + 1
};
// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
         ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32);
}
__device__ __forceinline__ uint64_t opaque(uint64_t v) {
  v = uniform64(v);
  asm("" : "+s"(v));
  return v;
}
__device__ __forceinline__ IntQ make_intq(uint64_t q) {
  return IntQ{opaque(0 - q), 4 * q, opaque(0 - 4 * q), opaque(4 * q + 1)};
}
__device__ __forceinline__ uint64_t mul_shoup_lazy4(uint64_t a, uint64_t w, uint64_t ws, const IntQ& c) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), s0 = (uint32_t)ws, s1 = (uint32_t)(ws >> 32);
  const uint32_t t1 = __umulhi(a0, s1), t2 = __umulhi(a1, s0);
  uint64_t h = (uint64_t)a1 * s1 + t1, cy;
  // h += t2 as a multiply-add (a 64-bit addition of a 32-bit word needs a zero half of its own)
  asm("v_mad_u64_u32 %0, %1, %2, 1, %0" : "+v"(h), "=s"(cy) : "v"(t2));
  // a w + h (-q) mod 2^64: the cross products' low words, then two multiply-adds
  const uint32_t w0 = (uint32_t)w, w1 = (uint32_t)(w >> 32), h0 = (uint32_t)h, h1 = (uint32_t)(h >> 32);
  const uint32_t n0 = (uint32_t)c.nq, n1 = (uint32_t)(c.nq >> 32);
  const uint32_t x = a0 * w1 + a1 * w0 + (h0 * n1 + h1 * n0);
  return (uint64_t)h0 * n0 + ((uint64_t)a0 * w0 + ((uint64_t)x << 32));
}
// -1 - v, kept apart from the addition that follows
__device__ __forceinline__ uint64_t cpl(uint64_t v) {
  v = ~v;
  asm("" : "+v"(v));
  return v;
}
// x in [0, 2m) -> [0, m) for m < 2^63, nm = -m: the difference's sign as a mask
__device__ __forceinline__ uint64_t csub(uint64_t x, uint64_t m, uint64_t nm) {
  const uint64_t d = x + nm;
  uint32_t k;
  asm("v_ashrrev_i32 %0, 31, %1" : "=v"(k) : "v"((uint32_t)(d >> 32)));
  return d + ((uint64_t)(k & (uint32_t)m) | ((uint64_t)(k & (uint32_t)(m >> 32)) << 32));
}
//   forward CT: x <- x mod 4q, t = y w in [0, 4q), (x, y) <- (x + t, x - t + 4q), both in [0, 8q);
//   inverse GS: (x, y) <- (x + y reduced to [0, 4q), (x - y + 4q) w in [0, 4q)).
// The forward transform's last pass and the inverse's scaling by 1/N return [0, q).
__device__ __forceinline__ void bf_fwd(uint64_t& x, uint64_t& y, uint64_t w, uint64_t ws, const IntQ& c) {
  const uint64_t a = csub(x, c.q4, c.nq4);
  const uint64_t t = mul_shoup_lazy4(y, w, ws, c);
  x = a + t;
  y = a + c.q4p1 + cpl(t);
}
__device__ __forceinline__ void bf_inv(uint64_t& x, uint64_t& y, uint64_t w, uint64_t ws, const IntQ& c) {
  const uint64_t d = x + c.q4p1 + cpl(y);
  x = csub(x + y, c.q4, c.nq4);
  y = mul_shoup_lazy4(d, w, ws, c);
}
// [0, 8q) -> [0, q)
__device__ __forceinline__ uint64_t canon8(uint64_t x, const IntQ& c, uint64_t q) {
  x = csub(x, c.q4, c.nq4);
  x = csub(x, 2 * q, 2 * c.nq);
  return csub(x, q, c.nq);
}

// fp64 butterflies: sums are brought back to (-q, q) on some stages only (red).  With values in
// (-c q, c q) a product lands in (-(1/2 + 3c/8) q, (1/2 + 3c/8) q) (fpmod.h's estimate error, q < 2^50),
// so from c = 1 a forward transform's four unreduced stages reach 1.9, 3.1, 4.8 and 7.1, and an
// inverse one's three reach 2, 4 and 8: every value an integer of at most 2^53, exact, and every
// product's operand below 8q.
__device__ __forceinline__ constexpr bool red_fwd(int st, int logc) { return (st & 3) == 3 || st == logc - 1; }
__device__ __forceinline__ constexpr bool red_inv(int st, int logc) { return (logc - 1 - st) % 3 == 2 || st == 0; }

template <bool FP>
__device__ __forceinline__ void bfly_fwd(uint64_t& x, uint64_t& y, uint64_t w, uint64_t ws, const IntQ& c, double qd,
                                         double qinv, bool red) {
  if (FP) {
    const double xd = b2f(x), v = fmulmod_s(b2f(y), b2f(w), qd, qinv);
    x = f2b(red ? sred(xd + v, qd, qinv) : xd + v);
    y = f2b(red ? sred(xd - v, qd, qinv) : xd - v);
  } else {
    bf_fwd(x, y, w, ws, c);
  }
}

template <bool FP>
__device__ __forceinline__ void bfly_inv(uint64_t& x, uint64_t& y, uint64_t w, uint64_t ws, const IntQ& c, double qd,
                                         double qinv, bool red) {
  if (FP) {
    const double xd = b2f(x), yd = b2f(y);
    x = f2b(red ? sred(xd + yd, qd, qinv) : xd + yd);
    y = f2b(fmulmod_s(red ? sred(xd - yd, qd, qinv) : xd - yd, b2f(w), qd, qinv));
  } else {
    bf_inv(x, y, w, ws, c);
  }
}

// Shape of one pass: sub-transforms of C points, TPC threads each, EPT points a thread.
template <int LOGC, int COLS>
struct PassGeo {
  static constexpr int C = 1 << LOGC;
  static constexpr int LT = LOGC / 2;
  static constexpr int TPC = 1 << LT;
  static constexpr int LE = LOGC - LT;
  static constexpr int EPT = 1 << LE;
  static constexpr int THREADS = TPC * COLS;
  // one pad word per EPT elements (row pass) or one group width per EPT rows
  // (column pass) keeps the contiguous-layout accesses off a single bank set
  static constexpr int LDS_WORDS = COLS * (C + TPC);
};

// f(integral_constant<int, i>) for i in [A, B).  A 512-point pass's stages are too much code for the
// compiler to unroll a loop over them, and a loop's elements and twiddles would lie in memory (784 bytes a
// lane; an integer transform of 8 limbs at N = 2^17 took 70 us that way, 23 us in registers).
template <int A, int B, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (A < B) {
    f(std::integral_constant<int, A>{});
    static_for<A + 1, B>(f);
  }
}
// groups that a thread's contiguous points touch at stage st (of those narrower than a thread's points), and
// at the stages from a to b
template <class G>
__device__ __forceinline__ constexpr int stage_groups(int st) {
  return G::EPT / (2 * (G::C >> (st + 1))) > 0 ? G::EPT / (2 * (G::C >> (st + 1))) : 1;
}
template <class G>
__device__ __forceinline__ constexpr int stage_groups(int a, int b) {
  int n = 0;
  for (int st = a; st < b; ++st) n += stage_groups<G>(st);
  return n;
}

// Row passes of one wave per workgroup: row_cols chunks of C words, so a barrier costs nothing.
template <int LOGC>
constexpr int row_cols() {
  return 64 / PassGeo<LOGC, 1>::TPC;
}

// A prime's twiddles: forward (psi) or inverse (ipsi) rows of the context's tables
struct Tw {
  const uint64_t* W;
  const uint64_t* Ws;
  const double* Wf;
  uint64_t q;
  double qd, qinv;
  IntQ c;
};
__device__ __forceinline__ Tw make_tw(const uint64_t* tw, const uint64_t* tws, const double* twf, uint64_t q,
                                      double qinv, int mi, int log_n) {
  const size_t o = (size_t)mi << log_n;
  return Tw{tw + o, tws + o, twf + o, q, (double)q, qinv, make_intq(q)};
}
// every prime's tables, for kernels that run stages of their own
struct TwTables {
  const uint64_t *psi, *psi_s, *ipsi, *ipsi_s;
  const double *psi_f, *ipsi_f;
  const Mod* mods;
};
inline TwTables tw_tables(const ckks_ctx* c) {
  return TwTables{c->t.psi, c->t.psi_s, c->t.ipsi, c->t.ipsi_s, c->t.psi_f, c->t.ipsi_f, c->t.mods};
}
// primes that take the fp64 residue arithmetic
__device__ __forceinline__ bool fp_prime(uint64_t q) { return q > (1ull << 49) && q < (1ull << 50); }

// A thread's part of a pass: row r of sub-transform `col` of the workgroup, which is column or
// chunk `unit` of the limb.
// Column pass: consecutive threads = consecutive columns (coalesced rows); row pass: consecutive
// threads = consecutive elements of one chunk.
template <int LOGC, int COLS, bool ROW>
struct Place {
  typedef PassGeo<LOGC, COLS> G;
  int col, r, unit;
  __device__ __forceinline__ Place(int tid, int block)
      : col(ROW ? tid / G::TPC : tid % COLS), r(ROW ? tid % G::TPC : tid / COLS), unit(block * COLS + col) {}
  // LDS word of element e of this unit
  __device__ __forceinline__ int sidx(int e) const {
    return ROW ? col * (G::C + G::TPC) + e + e / G::EPT : e * COLS + col + (e / G::EPT) * COLS;
  }
  // word of element e inside the limb
  __device__ __forceinline__ uint32_t gidx(int e, int log_n) const {
    return ROW ? (uint32_t)unit * G::C + e : ((uint32_t)e << (log_n - LOGC)) + unit;
  }
  // twiddle of group i at local stage st
  __device__ __forceinline__ int twi(int st, int i, int log_n) const {
    return ROW ? (1 << (log_n - LOGC + st)) + unit * (1 << st) + i : (1 << st) + i;
  }
};

// Forward stages of one sub-transform: x in the strided layout (element r + TPC u) on entry, in
// the contiguous layout (element r EPT + v) on return.  `s` is free on entry.
template <int LOGC, int COLS, bool ROW, bool FP, int E>
__device__ __forceinline__ void fwd_core(uint64_t (&x)[E], uint64_t* s,
                                         const Place<LOGC, COLS, ROW>& p, const Tw& t, int log_n) {
  typedef PassGeo<LOGC, COLS> G;
  constexpr int C = G::C, TPC = G::TPC, LE = G::LE, EPT = G::EPT;
  static_assert(E == EPT, "one thread's points");
  auto twv = [&](int k) { return FP ? f2b(t.Wf[k]) : t.W[k]; };
  auto tws = [&](int k) { return FP ? (uint64_t)0 : t.Ws[k]; };
  // stages 0..LE-1 (butterfly distance >= TPC) in registers
  {
    uint64_t w[EPT], ws[EPT];
#pragma unroll
    for (int st = 0; st < LE; ++st)
#pragma unroll
      for (int i = 0; i < (1 << st); ++i) {
        const int k = p.twi(st, i, log_n);
        w[(1 << st) + i - 1] = twv(k);
        ws[(1 << st) + i - 1] = tws(k);
      }
    static_for<0, LE>([&](auto stage) {
      constexpr int st = stage, tu = EPT >> (st + 1);
#pragma unroll
      for (int u = 0; u < EPT; ++u)
        if ((u & tu) == 0) {
          const int i = u / (2 * tu);
          bfly_fwd<FP>(x[u], x[u + tu], w[(1 << st) + i - 1], ws[(1 << st) + i - 1], t.c, t.qd, t.qinv,
                       red_fwd(st, LOGC));
        }
    });
  }
  // transpose to the contiguous layout
#pragma unroll
  for (int u = 0; u < EPT; ++u) s[p.sidx(p.r + TPC * u)] = x[u];
  __syncthreads();
#pragma unroll
  for (int v = 0; v < EPT; ++v) x[v] = s[p.sidx(p.r * EPT + v)];
  // stages LE..LOGC-1 (butterfly distance < TPC)
  {
    uint64_t w[EPT], ws[EPT];   // at most EPT - 1 twiddles in these stages
    int pos = 0;
#pragma unroll
    for (int st = LE; st < LOGC; ++st) {
      const int d = C >> (st + 1);
      const int ng = EPT / (2 * d) > 0 ? EPT / (2 * d) : 1;   // groups touched by this thread
#pragma unroll
      for (int gi = 0; gi < ng; ++gi) {
        const int k = p.twi(st, (p.r * EPT) / (2 * d) + gi, log_n);
        w[pos] = twv(k);
        ws[pos] = tws(k);
        ++pos;
      }
    }
    static_for<LE, LOGC>([&](auto stage) {
      constexpr int st = stage, d = C >> (st + 1), first = stage_groups<G>(LE, st);
#pragma unroll
      for (int v = 0; v < EPT; ++v)
        if ((v & d) == 0) {
          const int g = first + v / (2 * d);
          bfly_fwd<FP>(x[v], x[v + d], w[g], ws[g], t.c, t.qd, t.qinv, red_fwd(st, LOGC));
        }
    });
  }
}

// Inverse stages of one sub-transform: contiguous layout on entry, strided on return (not scaled
// by 1/N).  `s` is free on entry.
template <int LOGC, int COLS, bool ROW, bool FP, int E>
__device__ __forceinline__ void inv_core(uint64_t (&x)[E], uint64_t* s,
                                         const Place<LOGC, COLS, ROW>& p, const Tw& t, int log_n) {
  typedef PassGeo<LOGC, COLS> G;
  constexpr int C = G::C, TPC = G::TPC, LE = G::LE, EPT = G::EPT;
  static_assert(E == EPT, "one thread's points");
  auto twv = [&](int k) { return FP ? f2b(t.Wf[k]) : t.W[k]; };
  auto tws = [&](int k) { return FP ? (uint64_t)0 : t.Ws[k]; };
  // stages LOGC-1..LE (butterfly distance < TPC) in registers
  {
    uint64_t w[EPT], ws[EPT];   // at most EPT - 1 twiddles in these stages
    int pos = 0;
#pragma unroll
    for (int st = LOGC - 1; st >= LE; --st) {
      const int d = C >> (st + 1);
      const int ng = EPT / (2 * d) > 0 ? EPT / (2 * d) : 1;
#pragma unroll
      for (int gi = 0; gi < ng; ++gi) {
        const int k = p.twi(st, (p.r * EPT) / (2 * d) + gi, log_n);
        w[pos] = twv(k);
        ws[pos] = tws(k);
        ++pos;
      }
    }
    static_for<0, LOGC - LE>([&](auto stage) {
      constexpr int st = LOGC - 1 - stage, d = C >> (st + 1), first = stage_groups<G>(st + 1, LOGC);
#pragma unroll
      for (int v = 0; v < EPT; ++v)
        if ((v & d) == 0) {
          const int g = first + v / (2 * d);
          bfly_inv<FP>(x[v], x[v + d], w[g], ws[g], t.c, t.qd, t.qinv, red_inv(st, LOGC));
        }
    });
  }
  // transpose to the strided layout
#pragma unroll
  for (int v = 0; v < EPT; ++v) s[p.sidx(p.r * EPT + v)] = x[v];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < EPT; ++u) x[u] = s[p.sidx(p.r + TPC * u)];
  // stages LE-1..0 (butterfly distance >= TPC)
  {
    uint64_t w[EPT], ws[EPT];
#pragma unroll
    for (int st = 0; st < LE; ++st)
#pragma unroll
      for (int i = 0; i < (1 << st); ++i) {
        const int k = p.twi(st, i, log_n);
        w[(1 << st) + i - 1] = twv(k);
        ws[(1 << st) + i - 1] = tws(k);
      }
    static_for<0, LE>([&](auto stage) {
      constexpr int st = LE - 1 - stage, tu = EPT >> (st + 1);
#pragma unroll
      for (int u = 0; u < EPT; ++u)
        if ((u & tu) == 0) {
          const int i = u / (2 * tu);
          bfly_inv<FP>(x[u], x[u + tu], w[(1 << st) + i - 1], ws[(1 << st) + i - 1], t.c, t.qd, t.qinv,
                       red_inv(st, LOGC));
        }
    });
  }
}

// ---- column passes of eight points a thread ----------------------------------------------------
// A block of 16 columns (128-byte runs of a limb's rows) has TPC = C / 8 threads a column with 8
// elements each, so that four waves a SIMD fit and hide each other's waits (a fused ModUp of 13 ciphertexts at
// N = 2^16 took 82 us, with 16 elements a thread and two waves a SIMD 105 us).  The stages run in up to three layouts of a thread's elements:
//   A  r + TPC u                              the three widest butterflies;
//   B  (r / S) 8 S + r % S + S u, S = TPC / 8 the next three (TPC > 8; else B is C);
//   C  8 r + v                                the rest.
// A to B goes through LDS with one barrier; B to C stays within a wave (the S threads of a group
// times 16 columns are at most 64 lanes).  LDS is double buffered: the next transform's stores
// cannot meet the previous one's loads, which every wave has done before the barrier between.
constexpr int MID_COLS = 16;
template <int LOGC, int COLS = MID_COLS>
struct MidGeo {
  static constexpr int C = 1 << LOGC;
  static constexpr int EPT = 8;
  static constexpr int TPC = C / 8;
  static constexpr int S = TPC > 8 ? TPC / 8 : 1;
  static constexpr int THREADS = TPC * COLS;
  static constexpr int BUF = COLS * (C + C / 8);   // a pad row per eight spreads layout C over the banks
};
// LDS word of element e: (e + e / 8) COLS + column.  In every layout that is a base of the thread plus
// a constant of u (a layout's steps never carry the first element's remainder past a row of eight).
template <int LOGC, int COLS = MID_COLS>
struct MidPlace {
  typedef MidGeo<LOGC, COLS> G;
  int r, unit, e0b, sa, sb, sc;
  __device__ __forceinline__ MidPlace(int tid, int block)
      : r(tid / COLS), unit(block * COLS + tid % COLS), e0b((r / G::S) * (8 * G::S) + r % G::S) {
    const int col = tid % COLS;
    sa = (r + (r >> 3)) * COLS + col;
    sb = (e0b + (r / G::S) * G::S) * COLS + col;
    sc = 9 * r * COLS + col;
  }
  __device__ __forceinline__ int a(int u) const { return sa + (G::TPC * u + ((G::TPC * u) >> 3)) * COLS; }
  __device__ __forceinline__ int b(int u) const { return sb + (G::S * u + ((G::S * u) >> 3)) * COLS; }
  __device__ __forceinline__ int c(int v) const { return sc + v * COLS; }
  // word of element 8 r + v of a limb: v's part is the same for every thread
  __device__ __forceinline__ uint32_t word(int log_n) const { return ((uint32_t)(8 * r) << (log_n - LOGC)) + unit; }
  __device__ __forceinline__ size_t row(int v, int log_n) const { return (size_t)v << (log_n - LOGC); }
};
// twiddles of stages [S0, S1) on a thread's 8 elements, whose first is e0 and whose step is STEP;
// stage st pairs elements C >> (st + 1) apart
template <bool FP>
struct MidTw {
  uint64_t w[7], ws[FP ? 1 : 7];
};
template <int LOGC, bool FP, int S0, int S1, int STEP, bool UNIFORM>
__device__ __forceinline__ void mid_tw(MidTw<FP>& m, int e0, const Tw& t) {
  int n = 0;
#pragma unroll
  for (int st = S0; st < S1; ++st) {
    const int d = (1 << LOGC) >> (st + 1);
    const int ng = 4 / (d / STEP) > 0 ? 4 / (d / STEP) : 1;
#pragma unroll
    for (int g = 0; g < ng; ++g) {
      const int k = (1 << st) + e0 / (2 * d) + g;
      if (UNIFORM) {
        m.w[n] = FP ? f2b(cld(t.Wf + k)) : cld(t.W + k);
        if (!FP) m.ws[n] = cld(t.Ws + k);
      } else {
        m.w[n] = FP ? f2b(t.Wf[k]) : t.W[k];
        if (!FP) m.ws[n] = t.Ws[k];
      }
      ++n;
    }
  }
}
template <int LOGC, bool FP, bool INV, int S0, int S1, int STEP>
__device__ __forceinline__ void mid_stages(uint64_t (&x)[8], const MidTw<FP>& m, const Tw& t) {
#pragma unroll
  for (int i = S0; i < S1; ++i) {
    const int st = INV ? S1 - 1 - (i - S0) : i;
    const int du = ((1 << LOGC) >> (st + 1)) / STEP;   // the pair's distance in this thread's elements
    int n = 0;
    for (int s = S0; s < st; ++s) n += 4 / (((1 << LOGC) >> (s + 1)) / STEP) > 0 ? 4 / (((1 << LOGC) >> (s + 1)) / STEP) : 1;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if ((u & du) == 0) {
        const int g = n + u / (2 * du);
        if (INV)
          bfly_inv<FP>(x[u], x[u + du], m.w[g], FP ? 0 : m.ws[FP ? 0 : g], t.c, t.qd, t.qinv, red_inv(st, LOGC));
        else
          bfly_fwd<FP>(x[u], x[u + du], m.w[g], FP ? 0 : m.ws[FP ? 0 : g], t.c, t.qd, t.qinv, red_fwd(st, LOGC));
      }
  }
}
// the wave's own LDS words, stored by one lane and loaded by another: in program order
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// layout A -> layout C, forward stages; s: this transform's LDS buffer.  In fp64 each layout's
// twiddles are requested before the wait of the layout before it, `first` (layout B's, or C's when
// there is no B) before the map; the integer form's, twice as many registers, where they are used.
template <int LOGC, bool FP, int COLS>
__device__ __forceinline__ void mid_fwd_first(MidTw<FP>& m, const MidPlace<LOGC, COLS>& p, const Tw& t) {
  typedef MidGeo<LOGC, COLS> G;
  if (G::S > 1)
    mid_tw<LOGC, FP, 3, (G::S > 1 ? 6 : 3), G::S, false>(m, p.e0b, t);
  else
    mid_tw<LOGC, FP, 3, (G::S > 1 ? 3 : LOGC), 1, false>(m, 8 * p.r, t);
}
template <int LOGC, bool FP, int COLS>
__device__ __forceinline__ void mid_fwd(uint64_t (&x)[8], uint64_t* s, const MidPlace<LOGC, COLS>& p, const Tw& t,
                                        MidTw<FP>& first) {
  typedef MidGeo<LOGC, COLS> G;
  {
    MidTw<FP> a;
    mid_tw<LOGC, FP, 0, 3, G::TPC, true>(a, 0, t);
    mid_stages<LOGC, FP, false, 0, 3, G::TPC>(x, a, t);
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) s[p.a(u)] = x[u];
  __syncthreads();
  if (!FP) mid_fwd_first<LOGC, FP>(first, p, t);
  if (G::S > 1) {
    MidTw<FP> c;
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = s[p.b(u)];
    if (FP) mid_tw<LOGC, FP, 6, (G::S > 1 ? LOGC : 6), 1, false>(c, 8 * p.r, t);
    mid_stages<LOGC, FP, false, 3, (G::S > 1 ? 6 : 3), G::S>(x, first, t);
#pragma unroll
    for (int u = 0; u < 8; ++u) s[p.b(u)] = x[u];
    wave_order();
#pragma unroll
    for (int v = 0; v < 8; ++v) x[v] = s[p.c(v)];
    if (!FP) mid_tw<LOGC, FP, 6, (G::S > 1 ? LOGC : 6), 1, false>(c, 8 * p.r, t);
    mid_stages<LOGC, FP, false, 6, (G::S > 1 ? LOGC : 6), 1>(x, c, t);
  } else {
#pragma unroll
    for (int v = 0; v < 8; ++v) x[v] = s[p.c(v)];
    mid_stages<LOGC, FP, false, 3, (G::S > 1 ? 3 : LOGC), 1>(x, first, t);
  }
}
// layout C -> layout A, inverse stages
template <int LOGC, bool FP, int COLS>
__device__ __forceinline__ void mid_inv(uint64_t (&x)[8], uint64_t* s, const MidPlace<LOGC, COLS>& p, const Tw& t) {
  typedef MidGeo<LOGC, COLS> G;
  constexpr int SC = G::S > 1 ? 6 : 3;   // first stage of layout C
  MidTw<FP> c, b;
  mid_tw<LOGC, FP, SC, LOGC, 1, false>(c, 8 * p.r, t);
  if (FP && G::S > 1) mid_tw<LOGC, FP, 3, SC, G::S, false>(b, p.e0b, t);
  mid_stages<LOGC, FP, true, SC, LOGC, 1>(x, c, t);
#pragma unroll
  for (int v = 0; v < 8; ++v) s[p.c(v)] = x[v];
  if (G::S > 1) {
    wave_order();
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = s[p.b(u)];
    if (!FP) mid_tw<LOGC, FP, 3, SC, G::S, false>(b, p.e0b, t);
    mid_stages<LOGC, FP, true, 3, SC, G::S>(x, b, t);
#pragma unroll
    for (int u = 0; u < 8; ++u) s[p.b(u)] = x[u];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 8; ++u) x[u] = s[p.a(u)];
  MidTw<FP> a;
  mid_tw<LOGC, FP, 0, 3, G::TPC, true>(a, 0, t);
  mid_stages<LOGC, FP, true, 0, 3, G::TPC>(x, a, t);
}

// A forward column pass whose input a functor makes: src.load<LOGC, FP>(x, s, p, limb's modulus index, Mod,
// poly, t, log_n) fills x in layout A, in (-q, q) (fp64) or [0, 8q).  It may use the LDS buffer s if each thread
// ends with its own words of layout A (which are then its to overwrite).  Limb i of polynomial z goes to out + z * stride + i N, half transformed.
template <int LOGC, int COLS, class S>
__global__ __launch_bounds__((1 << LOGC) / 8 * COLS) void k_src_cols(uint64_t* __restrict__ out, size_t stride, S src,
                                                                        LimbMap map, TwTables tt, int log_n) {
  typedef MidGeo<LOGC, COLS> G;
  __shared__ uint64_t s[G::BUF];
  const int i = blockIdx.y, z = blockIdx.z, mi = lm_mod(map, i);
  const Mod m = cld(tt.mods + mi);
  const MidPlace<LOGC, COLS> p(threadIdx.x, blockIdx.x);
  const Tw t = make_tw(tt.psi, tt.psi_s, tt.psi_f, m.q, m.qinv, mi, log_n);
  uint64_t* a = out + z * stride + ((size_t)i << log_n) + p.word(log_n);
  uint64_t x[8];
  auto run = [&](auto fp) {
    constexpr bool FP = decltype(fp)::value;
    src.template load<LOGC, FP>(x, s, p, mi, m, z, t, log_n);
    MidTw<FP> first;
    if (FP) mid_fwd_first<LOGC, FP>(first, p, t);
    mid_fwd<LOGC, FP>(x, s, p, t, first);
  };
  if (fp_prime(m.q))
    run(std::integral_constant<bool, true>{});
  else
    run(std::integral_constant<bool, false>{});
#pragma unroll
  for (int v = 0; v < 8; ++v) (a + p.row(v, log_n))[0] = x[v];
}
template <class S>
static void src_cols(ckks_ctx* c, uint64_t* out, size_t stride, const S& src, int n_limbs, LimbMap map, int n_polys) {
  const TwTables tt = tw_tables(c);
  // half the columns a workgroup (64-byte runs) where there would be less than two workgroups a CU: one encryption's
  // 224 workgroups of 512 threads at N = 2^16 took 13.5 us, 448 of 256 take 12.1
  const int lc = ntt_mid_log(c);
  const bool narrow = lc >= 6 && (size_t)((c->N >> lc) / MID_COLS) * n_limbs * n_polys < 512;
#define Y(LC, CO)                                                                                                   \
  hipLaunchKernelGGL((k_src_cols<LC, CO, S>), dim3((c->N >> LC) / (CO), n_limbs, n_polys), dim3((1 << LC) / 8 * (CO)), 0, \
                     c->stream, out, stride, src, map, tt, c->log_n)
#define X(LC)           \
  if (narrow)           \
    Y(LC, MID_COLS / 2); \
  else                  \
    Y(LC, MID_COLS)
  switch (lc) {
    case 4: Y(4, 2 * MID_COLS); break;   // two threads a column: 32 of them are a wave
    case 5: Y(5, MID_COLS); break;
    case 6: X(6); break;
    case 7: X(7); break;
    case 8: X(8); break;
    default: FICGCN_THROW(EINVAL_, "unsupported ring degree");
  }
#undef X
#undef Y
  HIPCHECK(hipGetLastError());
}

}  // namespace ficgcn
