// Tables of the canonical embedding (host, FP64); encode_gpu.hip evaluates it both ways.
//
// Slot j of m(X) in Z[X]/(X^N+1) is m(zeta^(5^j)), zeta = exp(i pi / N); the
// conjugate slots sit at zeta^(-5^j).  Encoding evaluates the inverse embedding with one
// complex FFT over the N odd powers of zeta:
//   v_s = value at zeta^(2s+1),  m_i = Re(exp(-i pi i / N) FFT(v)_i) / N.
#include <cmath>
#include <complex>
#include <map>
#include <mutex>
#include <vector>

#include "internal.h"

namespace ficgcn {

typedef std::complex<double> cd;

// exp(-2 pi i k / n) for k < n/2, and exp(-i pi i / n) for i < n; cached per n
struct FftTables {
  std::vector<cd> root, twist;
};

static const FftTables& tables(size_t n) {
  static std::mutex mu;
  static std::map<size_t, FftTables> cache;
  std::lock_guard<std::mutex> g(mu);
  auto it = cache.find(n);
  if (it != cache.end()) return it->second;
  FftTables t;
  t.root.resize(n / 2);
  for (size_t k = 0; k < n / 2; ++k) t.root[k] = cd(std::cos(2 * M_PI * k / n), -std::sin(2 * M_PI * k / n));
  t.twist.resize(n);
  for (size_t i = 0; i < n; ++i) t.twist[i] = cd(std::cos(M_PI * i / n), -std::sin(M_PI * i / n));
  return cache[n] = t;
}

// 5^j mod 2N for the N/2 slots, cached per N
static const std::vector<uint32_t>& slot_exponents(int N) {
  static std::mutex mu;
  static std::map<int, std::vector<uint32_t>> cache;
  std::lock_guard<std::mutex> g(mu);
  auto it = cache.find(N);
  if (it != cache.end()) return it->second;
  std::vector<uint32_t> r(N / 2);
  uint64_t x = 1;
  for (int j = 0; j < N / 2; ++j) {
    r[j] = (uint32_t)x;
    x = x * 5 % (2 * (uint64_t)N);
  }
  return cache[N] = r;
}

void encode_tables(int N, std::vector<double>& root, std::vector<double>& twist, std::vector<uint32_t>& pos,
                   std::vector<uint32_t>& src) {
  const FftTables& T = tables(N);
  const std::vector<uint32_t>& r = slot_exponents(N);
  root.resize((size_t)N);
  for (int k = 0; k < N / 2; ++k) {
    root[2 * k] = T.root[k].real();
    root[2 * k + 1] = T.root[k].imag();
  }
  twist.resize((size_t)2 * N);
  for (int i = 0; i < N; ++i) {
    twist[2 * i] = T.twist[i].real();
    twist[2 * i + 1] = T.twist[i].imag();
  }
  pos.resize((size_t)N / 2);
  src.resize((size_t)N);
  for (int j = 0; j < N / 2; ++j) {
    pos[j] = (r[j] - 1) / 4;
    src[(r[j] - 1) / 2] = 2 * (uint32_t)j;
    src[(2 * (uint32_t)N - r[j] - 1) / 2] = 2 * (uint32_t)j + 1;
  }
}

}  // namespace ficgcn
