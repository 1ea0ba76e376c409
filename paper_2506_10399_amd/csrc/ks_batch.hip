// Batched hybrid key switching and batched ciphertext kernels.
//
// A batch holds R key switches at one level whose inputs come from U
// distinct source polynomials (U = 1 when every rotation of one ciphertext
// is hoisted on its ModUp; U = R when each ciphertext is switched once, as
// for relinearising a layer).  Each stage is one launch over the batch:
//   ModUp  : inverse NTT of the U sources, fast base conversion of every
//            digit of every source, forward NTT of the extended limbs (for one or
//            two special primes the conversion runs inside the transforms' column
//            passes, ntt_fused.hip; the same for ModDown and the rescales);
//   inner  : acc_r = sum_d sigma_{g_r}(D_{src(r),d}) * key_{r,d}   (both components);
//   ModDown: inverse NTT of the P limbs of every acc_r, rounded conversion
//            to Q_l, forward NTT, then the grouped final step
//            out_grp (+)= sum_r ((acc_r - conv_r) * P^-1 + add_r) [(.) pt_r].
// Every switch is the same exact modular computation as a single key
// switch (ModUp, automorphism on the digits, inner product, ModDown with
// rounding), so the words equal those of R separate switches.  The
// grouped final step replaces "write R switched ciphertexts, read them
// back for a masked sum" by one read of acc and conv per switch.
#include <algorithm>
#include <cstring>
#include <map>
#include <numeric>
#include <tuple>

#include "fpmod.h"
#include "ks_batch.h"
#include "ks_common.h"
#include "ntt_dev.h"
#include "ntt_fused.h"

namespace ficgcn {

void zero_fill(ckks_ctx* c, uint64_t* p, size_t words);

constexpr int KB = 256;

__device__ const uint64_t k_one_word = 1;

// tmp[u] = sources[u] (l1 limbs)
__global__ void k_gather(uint64_t* __restrict__ tmp, const uint64_t* const* __restrict__ src, int l1, int log_n) {
  const size_t N = (size_t)1 << log_n;
  const size_t j = blockIdx.x * (size_t)KB + threadIdx.x;
  const int i = blockIdx.y, u = blockIdx.z;
  tmp[((size_t)u * l1 + i) * N + j] = gld(src[u] + (size_t)i * N + j);
}

struct DigitTables {
  enum { MAX = 32 };
  const uint64_t* tab[MAX];   // [n_src] hat_inv, [n_src] Shoup, [n_dst][n_src] hat mod dst
  const int* idx[MAX];        // [n_src] source moduli, then [n_dst] destination moduli
  int n_src[MAX];
  int n_dst[MAX];
};

// Digit d of source u: the digit's residues (coefficient form, in tmp)
// converted to every other prime of Q_l and P; the digit's own limbs are
// the source limbs in evaluation form.
__global__ void k_modup_conv(const uint64_t* __restrict__ tmp, const uint64_t* const* __restrict__ src,
                             uint64_t* __restrict__ D, DigitTables dt, int alpha, int l1, int ext, int nd, int L,
                             int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const size_t j = blockIdx.x * (size_t)KB + threadIdx.x;
  const int d = blockIdx.y, u = blockIdx.z;
  const uint64_t* tab = dt.tab[d];
  const int* idx = dt.idx[d];
  const int ns = dt.n_src[d], ndst = dt.n_dst[d];
  const uint64_t* s = tmp + ((size_t)u * l1 + (size_t)d * alpha) * N;
  const uint64_t* own = src[u] + (size_t)d * alpha * N;
  uint64_t* Dd = D + ((size_t)u * nd + d) * ext * N;
  uint64_t y[8];
  for (int t = 0; t < ns; ++t) {
    const uint64_t b = mods[idx[t]].q;
    y[t] = mul_shoup(s[t * N + j], tab[t], tab[ns + t], b);
    Dd[((size_t)d * alpha + t) * N + j] = gld(own + t * N + j);
  }
  const uint64_t* hm = tab + 2 * ns;
  for (int k = 0; k < ndst; ++k) {
    const int m = idx[ns + k];
    const Mod md = mods[m];
    u128 acc = 0;
    for (int t = 0; t < ns; ++t) acc += (u128)y[t] * hm[k * ns + t];
    const int pos = m < L ? m : m - L + l1;
    Dd[(size_t)pos * N + j] = reduce128(acc, md);
  }
}

// acc[r][c][i] = sum_d D_{src(r),d}[i][sigma_g(j)] * key_r[d][c][m(i)][j]
__global__ void k_keymac_batch(uint64_t* __restrict__ acc, const uint64_t* __restrict__ D,
                               const KSJob* __restrict__ jobs, int nd, int ext, int l1, int L, int n_mod, int log_n,
                               const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const uint32_t j = blockIdx.x * KB + threadIdx.x;
  const int i = blockIdx.y, r = blockIdx.z;
  const KSJob jb = jobs[r];
  const int m = i < l1 ? i : i - l1 + L;
  const uint32_t jj = jb.g == 1 ? j : auto_idx(j, jb.g, log_n);
  const uint64_t* Du = D + (size_t)jb.src * nd * ext * N;
  u128 s0 = 0, s1 = 0;
  for (int d = 0; d < nd; ++d) {
    const u128 x = Du[((size_t)d * ext + i) * N + jj];
    s0 += x * gld(jb.key + (((size_t)d * 2 + 0) * n_mod + m) * N + j);
    s1 += x * gld(jb.key + (((size_t)d * 2 + 1) * n_mod + m) * N + j);
  }
  const Mod md = mods[m];
  acc[(((size_t)r * 2 + 0) * ext + i) * N + j] = reduce128(s0, md);
  acc[(((size_t)r * 2 + 1) * ext + i) * N + j] = reduce128(s1, md);
}

// The same inner products with jobs taken in runs that share one key (and Galois element):
// a thread reads its key words once and applies them to every job of its run (the rotations
// of several ciphertexts by one step), so the key streams from HBM once per run.
constexpr int KR_MAXD = 8;   // digits held in registers (the kernels are instantiated per digit count)
template <int ND>
__global__ void k_keymac_runs(uint64_t* __restrict__ acc, const uint64_t* __restrict__ D,
                              const KSJob* __restrict__ jobs, const int* __restrict__ run_start, int ext, int l1,
                              int L, int n_mod, int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const uint32_t j = blockIdx.x * KB + threadIdx.x;
  const int i = blockIdx.y;
  const int r0 = run_start[blockIdx.z], r1 = run_start[blockIdx.z + 1];
  const KSJob j0 = jobs[r0];
  const int m = i < l1 ? i : i - l1 + L;
  const uint32_t jj = j0.g == 1 ? j : auto_idx(j, j0.g, log_n);
  uint64_t k0[ND], k1[ND];
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    k0[d] = gld(j0.key + (((size_t)d * 2 + 0) * n_mod + m) * N + j);
    k1[d] = gld(j0.key + (((size_t)d * 2 + 1) * n_mod + m) * N + j);
  }
  const Mod md = mods[m];
  for (int r = r0; r < r1; ++r) {
    const uint64_t* Du = D + (size_t)jobs[r].src * ND * ext * N;
    u128 s0 = 0, s1 = 0;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      const u128 x = Du[((size_t)d * ext + i) * N + jj];
      s0 += x * k0[d];
      s1 += x * k1[d];
    }
    acc[(((size_t)r * 2 + 0) * ext + i) * N + j] = reduce128(s0, md);
    acc[(((size_t)r * 2 + 1) * ext + i) * N + j] = reduce128(s1, md);
  }
}

// runs of consecutive jobs with one key and Galois element; host side
static std::vector<int> key_runs(const std::vector<KSJob>& jobs) {
  std::vector<int> start;
  for (size_t r = 0; r < jobs.size(); ++r)
    if (r == 0 || jobs[r].key != jobs[r - 1].key || jobs[r].g != jobs[r - 1].g) start.push_back((int)r);
  start.push_back((int)jobs.size());
  return start;
}

// conv[z][i] = FastBConv_{P -> q_i}([acc_P + floor(P/2)]) - floor(P/2)   (coefficient form)
__global__ void k_moddown_conv_batch(const uint64_t* __restrict__ acc, int ext, int l1, const int* __restrict__ src_mod,
                                     const int* __restrict__ dst_mod, int ns, const uint64_t* __restrict__ table,
                                     MDK k, uint64_t* __restrict__ conv, int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const size_t j = blockIdx.x * (size_t)KB + threadIdx.x;
  const int z = blockIdx.y;   // r * 2 + component
  const uint64_t* ap = acc + ((size_t)z * ext + l1) * N;
  uint64_t y[8];
  for (int t = 0; t < ns; ++t) {
    const uint64_t b = mods[src_mod[t]].q;
    const uint64_t x = add_mod(ap[t * N + j], k.hP[t], b);
    y[t] = mul_shoup(x, table[t], table[ns + t], b);
  }
  const uint64_t* hm = table + 2 * ns;
  for (int d = 0; d < l1; ++d) {
    const Mod md = mods[dst_mod[d]];
    u128 a = 0;
    for (int t = 0; t < ns; ++t) a += (u128)y[t] * hm[d * ns + t];
    conv[((size_t)z * l1 + d) * N + j] = sub_mod(reduce128(a, md), k.hQ[d], md.q);
  }
}

struct GroupDesc {
  uint64_t* out;   // [2][l+1][N]
  int start, end;  // job range within the chunk
  int accumulate;
  int pad;
};

__global__ void k_ks_final(const uint64_t* __restrict__ acc, const uint64_t* __restrict__ conv, int ext, int l1, MDK k,
                           const KSJob* __restrict__ jobs, const GroupDesc* __restrict__ groups, int log_n,
                           const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const uint32_t j = blockIdx.x * KB + threadIdx.x;
  const int i = blockIdx.y;
  const int comp = blockIdx.z & 1;
  const GroupDesc gd = groups[blockIdx.z >> 1];
  const Mod md = mods[i];
  const uint64_t q = md.q;
  const size_t o = ((size_t)comp * l1 + i) * N + j;
  uint64_t a = gd.accumulate ? gld(gd.out + o) : 0;
  u128 s = 0;
  int cnt = 0;
  for (int r = gd.start; r < gd.end; ++r) {
    const KSJob jb = jobs[r];
    uint64_t v = sub_mod(acc[(((size_t)r * 2 + comp) * ext + i) * N + j],
                         conv[(((size_t)r * 2 + comp) * l1 + i) * N + j], q);
    v = mul_shoup(v, k.pinv[i], k.pinv_s[i], q);
    if (comp == 0 && jb.add0) v = add_mod(v, gld(jb.add0 + (size_t)i * N + (jb.g == 1 ? j : auto_idx(j, jb.g, log_n))), q);
    if (comp == 1 && jb.add1) v = add_mod(v, gld(jb.add1 + (size_t)i * N + j), q);
    if (jb.pt) {
      s += (u128)v * gld(jb.pt + (size_t)i * N + j);
      if (++cnt == 8) {
        a = add_mod(a, reduce128(s, md), q);
        s = 0;
        cnt = 0;
      }
    } else {
      a = add_mod(a, v, q);
    }
  }
  gst(gd.out + o, add_mod(a, reduce128(s, md), q));
}

enum { S_KB_TMP = 50, S_KB_D, S_KB_ACC, S_KB_CONV, S_KB_JOBS, S_TB_JOBS, S_RS_PTR, S_RS_LAST, S_RS_D, S_GM_TERMS };

// Device copies of a launch group's tables, in one transfer (each on a 16-byte boundary)
template <typename... T>
static std::tuple<T*...> upload(ckks_ctx* c, int slot, const std::vector<T>&... v) {
  size_t bytes = 0;
  const size_t at[] = {[&](size_t n) {
    const size_t o = bytes;
    bytes += (n + 15) & ~(size_t)15;
    return o;
  }(v.size() * sizeof(T))...};
  std::vector<uint8_t> h(bytes);
  size_t k = 0;
  (void)std::initializer_list<int>{((v.empty() ? (void)0 : (void)std::memcpy(h.data() + at[k], v.data(), v.size() * sizeof(T))), ++k, 0)...};
  uint8_t* d = (uint8_t*)dev_table(c, slot, h.data(), bytes);
  k = 0;
  return std::tuple<T*...>{(T*)(d + at[k++])...};
}

// ModUp of a batch's sources (device table of U polynomials [l1][N]) into D [U][nd][ext][N]
static void modup_batch(ckks_ctx* c, int level, const uint64_t* const* sd, int U, uint64_t* tmp, uint64_t* D) {
  if (fused_basis(c)) {
    modup_polys(c, level, sd, nullptr, U, tmp, D);
    return;
  }
  const size_t N = c->N;
  const int l1 = level + 1, ext = l1 + c->alpha;
  const int nd = (l1 + c->alpha - 1) / c->alpha;
  DigitTables dt{};
  for (int d = 0; d < nd; ++d) {
    const BConv& bc = get_modup(c, level, d);
    dt.tab[d] = bc.dev;
    dt.idx[d] = bc.idx;
    dt.n_src[d] = bc.n_src;
    dt.n_dst[d] = bc.n_dst;
  }
  hipLaunchKernelGGL(k_gather, dim3(N / KB, l1, U), dim3(KB), 0, c->stream, tmp, sd, l1, c->log_n);
  HIPCHECK(hipGetLastError());
  ntt_inv(c, tmp, l1, lm_q(l1), U, (size_t)l1 * N);
  hipLaunchKernelGGL(k_modup_conv, dim3(N / KB, nd, U), dim3(KB), 0, c->stream, tmp, sd, D, dt, c->alpha, l1, ext, nd,
                     c->L, c->log_n, c->t.mods);
  HIPCHECK(hipGetLastError());
  // every extended limb to evaluation form except each digit's own limbs
  ntt_fwd(c, D, ext, lm_ext(level, c->L), U * nd, (size_t)ext * N, c->alpha, l1);
}

// ModDown's conversion of Z accumulators [ext][N]: conv [Z][l1][N] in evaluation form
static void moddown_conv_batch(ckks_ctx* c, int level, uint64_t* acc, int Z, const MDK& k, uint64_t* conv) {
  if (fused_basis(c)) {
    moddown_polys(c, level, acc, Z, conv, true);
    return;
  }
  const size_t N = c->N;
  const int l1 = level + 1, ext = l1 + c->alpha;
  const BConv& md = get_moddown(c, level);
  ntt_inv(c, acc + (size_t)l1 * N, c->alpha, LimbMap{c->L, 1 << 30, 0}, Z, (size_t)ext * N);
  hipLaunchKernelGGL(k_moddown_conv_batch, dim3(N / KB, Z), dim3(KB), 0, c->stream, acc, ext, l1, md.idx,
                     md.idx + md.n_src, md.n_src, (const uint64_t*)md.dev, k, conv, c->log_n, c->t.mods);
  HIPCHECK(hipGetLastError());
  ntt_fwd(c, conv, l1, lm_q(l1), Z, (size_t)l1 * N);
}

// scratch bound of one chunk of a key-switch batch
static constexpr size_t KS_BUDGET = (size_t)3 << 30;

void keyswitch_batch(ckks_ctx* c, int level, const std::vector<const uint64_t*>& sources,
                     const std::vector<KSJob>& jobs, const std::vector<uint64_t*>& outs, bool accumulate) {
  const size_t N = c->N;
  const int l1 = level + 1, ext = l1 + c->alpha;
  const int nd = (l1 + c->alpha - 1) / c->alpha;
  const int n_grp = (int)outs.size();
  if (c->alpha > 8 || l1 > 64 || nd > DigitTables::MAX) FICGCN_THROW(EINVAL_, "too many primes");
  for (size_t r = 0; r < jobs.size(); ++r) {
    const KSJob& jb = jobs[r];
    if (jb.src < 0 || jb.src >= (int)sources.size() || !sources[jb.src] || !jb.key || jb.grp < 0 || jb.grp >= n_grp ||
        !outs[jb.grp] || (r && jobs[r - 1].grp > jb.grp))
      FICGCN_THROW(EINVAL_, "bad key-switch job");
  }
  ProfScope ps(c, "ks_batch");
  const size_t per_job = (size_t)2 * (ext + l1) * N * 8;
  const size_t per_src = (size_t)(nd * ext + l1) * N * 8;
  std::vector<char> touched(n_grp, 0);
  const MDK& k = c->mdk[level];
  size_t a = 0;
  while (a < jobs.size()) {
    // chunk [a, b): sources remapped to a dense local list
    std::vector<int> local(sources.size(), -1);
    std::vector<const uint64_t*> srcs;
    std::vector<KSJob> cj;
    size_t b = a, bytes = 0;
    while (b < jobs.size()) {
      const bool new_src = local[jobs[b].src] < 0;
      const size_t add = per_job + (new_src ? per_src : 0);
      if (b > a && bytes + add > KS_BUDGET) break;
      bytes += add;
      if (new_src) {
        local[jobs[b].src] = (int)srcs.size();
        srcs.push_back(sources[jobs[b].src]);
      }
      KSJob j = jobs[b];
      j.src = local[j.src];
      cj.push_back(j);
      ++b;
    }
    // groups of the chunk (contiguous since jobs are sorted by group)
    std::vector<GroupDesc> gds;
    for (size_t r = 0; r < cj.size(); ++r) {
      const int g = cj[r].grp;
      if (gds.empty() || r == 0 || cj[r - 1].grp != g) {
        gds.push_back(GroupDesc{outs[g], (int)r, (int)r + 1, (accumulate || touched[g]) ? 1 : 0, 0});
        touched[g] = 1;
      } else {
        gds.back().end = (int)r + 1;
      }
    }
    const int U = (int)srcs.size(), R = (int)cj.size();
    // one unmasked switch per output: the last step is part of the transform before it
    std::vector<FinalJob> finals;
    bool single = fused_basis(c) && gds.size() == cj.size();
    for (const KSJob& jb : cj) single = single && !jb.pt;
    if (single)
      for (int r = 0; r < R; ++r)
        finals.push_back(FinalJob{gds[r].out, cj[r].add0, cj[r].add1, cj[r].g, gds[r].accumulate, 0});
    std::vector<int> runs = key_runs(cj);
    const int n_runs = (int)runs.size() - 1;
    const auto [jd, sd, gd, fd, rd] = upload(c, S_KB_JOBS, cj, srcs, gds, finals, runs);
    uint64_t* tmp = (uint64_t*)dev_scratch(c, S_KB_TMP, (size_t)U * l1 * N * 8);
    uint64_t* D = (uint64_t*)dev_scratch(c, S_KB_D, (size_t)U * nd * ext * N * 8);
    uint64_t* acc = (uint64_t*)dev_scratch(c, S_KB_ACC, (size_t)R * 2 * ext * N * 8);
    uint64_t* conv = (uint64_t*)dev_scratch(c, S_KB_CONV, (size_t)R * 2 * l1 * N * 8);
    {
      ProfScope pm(c, "modup");
      modup_batch(c, level, sd, U, tmp, D);
    }
    {
      ProfScope pk(c, "keymac");
      if (n_runs < R && nd <= KR_MAXD) {   // some jobs share a key: each key read once per run
        const dim3 grid(N / KB, ext, n_runs);
#define KR_LAUNCH(NDV)                                                                                          \
  hipLaunchKernelGGL(k_keymac_runs<NDV>, grid, dim3(KB), 0, c->stream, acc, D, jd, rd, ext, l1, c->L, c->n_mod(), \
                     c->log_n, c->t.mods)
        switch (nd) {
          case 1: KR_LAUNCH(1); break;
          case 2: KR_LAUNCH(2); break;
          case 3: KR_LAUNCH(3); break;
          case 4: KR_LAUNCH(4); break;
          case 5: KR_LAUNCH(5); break;
          case 6: KR_LAUNCH(6); break;
          case 7: KR_LAUNCH(7); break;
          default: KR_LAUNCH(8);
        }
#undef KR_LAUNCH
      } else {
        hipLaunchKernelGGL(k_keymac_batch, dim3(N / KB, ext, R), dim3(KB), 0, c->stream, acc, D, jd, nd, ext, l1,
                           c->L, c->n_mod(), c->log_n, c->t.mods);
      }
      HIPCHECK(hipGetLastError());
    }
    {
      ProfScope pd(c, "moddown");
      if (finals.empty()) {
        moddown_conv_batch(c, level, acc, 2 * R, k, conv);
        hipLaunchKernelGGL(k_ks_final, dim3(N / KB, l1, 2 * gds.size()), dim3(KB), 0, c->stream, acc, conv, ext, l1,
                           k, jd, gd, c->log_n, c->t.mods);
        HIPCHECK(hipGetLastError());
      } else {
        moddown_polys(c, level, acc, 2 * R, conv, false);
        moddown_final(c, level, acc, conv, fd, FinalJob{}, R);
      }
    }
    a = b;
  }
  if (!accumulate)
    for (int g = 0; g < n_grp; ++g)
      if (!touched[g]) zero_fill(c, outs[g], (size_t)2 * l1 * N);
}

// ---- masked sums of key switches before one ModDown (double hoisting) ---------

struct MaskGroup {
  int start, end;   // job range (all jobs of the batch, sorted by group)
};

// The key inner products of a group's jobs and their masked sum in one pass:
// per job r, acc_r[c][i] = sum_d D_{src(r),d}[i][sigma_g(j)] * key_r[d][c][m(i)][j]
// (reduced), then A[c][i] += acc_r[c][i] (.) pt_r[i] (or + acc_r without a
// mask), both components per thread.  acc_r is never stored: the sums are
// those of the batched key inner product followed by a masked sum of its
// outputs, in the same order.
__global__ void k_keymac_masked(const uint64_t* __restrict__ D, const KSJob* __restrict__ jobs,
                                const GroupDesc* __restrict__ groups, int nd, int ext, int l1, int L, int n_mod,
                                int log_n, int n_groups, int xcd_order, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  // xcd_order: the groups of one coefficient block run back to back on one XCD
  // (blocks go round-robin over the 8 XCDs by linear id), so the keys the
  // groups share (one per shift) are read into that XCD's L2 once
  int jb, gi;
  if (xcd_order) {
    const int b = blockIdx.x, idx = b >> 3;
    jb = (b & 7) + 8 * (idx / n_groups);
    gi = idx % n_groups;
  } else {
    jb = blockIdx.x;
    gi = blockIdx.z;
  }
  const uint32_t j = (uint32_t)jb * KB + threadIdx.x;
  const int i = blockIdx.y;
  const GroupDesc gd = groups[gi];
  const int m = i < l1 ? i : i - l1 + L;
  const Mod md = mods[m];
  uint64_t* a0 = gd.out + (size_t)i * N + j;              // gd.out: this group's A
  uint64_t* a1 = gd.out + ((size_t)ext + i) * N + j;
  uint64_t v0 = gld(a0), v1 = gld(a1);
  u128 t0 = 0, t1 = 0;
  int cnt = 0;
  for (int r = gd.start; r < gd.end; ++r) {
    const KSJob jb = jobs[r];
    const uint32_t jj = jb.g == 1 ? j : auto_idx(j, jb.g, log_n);
    const uint64_t* Du = D + (size_t)jb.src * nd * ext * N;
    u128 s0 = 0, s1 = 0;
    for (int d = 0; d < nd; ++d) {
      const u128 x = Du[((size_t)d * ext + i) * N + jj];
      s0 += x * gld(jb.key + (((size_t)d * 2 + 0) * n_mod + m) * N + j);
      s1 += x * gld(jb.key + (((size_t)d * 2 + 1) * n_mod + m) * N + j);
    }
    const uint64_t x0 = reduce128(s0, md), x1 = reduce128(s1, md);
    if (jb.pt) {
      const uint64_t p = gld(jb.pt + (size_t)i * N + j);
      t0 += (u128)x0 * p;
      t1 += (u128)x1 * p;
    } else {
      t0 += x0;
      t1 += x1;
    }
    if (++cnt == 8) {
      v0 = add_mod(v0, reduce128(t0, md), md.q);
      v1 = add_mod(v1, reduce128(t1, md), md.q);
      t0 = 0;
      t1 = 0;
      cnt = 0;
    }
  }
  gst(a0, add_mod(v0, reduce128(t0, md), md.q));
  gst(a1, add_mod(v1, reduce128(t1, md), md.q));
}

// A + B 2^25 + C 2^50 mod q in [0, q) for a prime of the fp64 range.  A word v = v1 2^32 + v0 below 2^63
// comes back as v1 2^32 (an exact double, its quotient by q below 2^14) brought to (-q, q), plus v0.
__device__ __forceinline__ uint64_t fold25_fp(uint64_t A, uint64_t B, uint64_t C, double qd, double qinv, const Fold25& f) {
  auto part = [&](uint64_t v) {
    return sred((double)(uint32_t)(v >> 32) * 4294967296.0, qd, qinv) + (double)(uint32_t)v;
  };
  const double s = part(A) + (fmulmod_s(part(B), (double)f.r25, qd, qinv) + fmulmod_s(part(C), (double)f.r50, qd, qinv));
  return from_fbits(f2b(canon(sred(s, qd, qinv), qd)));
}
// the same for any prime below 2^50, each part lazily to [0, 4q)
__device__ __forceinline__ uint64_t fold25_int(uint64_t A, uint64_t B, uint64_t C, uint64_t q, const IntQ& iq,
                                               const Fold25& f) {
  const uint64_t v = mul_shoup_lazy4(A, 1, f.one_s, iq) + mul_shoup_lazy4(B, f.r25, f.r25_s, iq);
  return canon8(csub(v, iq.q4, iq.nq4) + mul_shoup_lazy4(C, f.r50, f.r50_s, iq), iq, q);
}
constexpr uint32_t M25 = (1u << 25) - 1;

// ---- the same rotations and masks for many outputs ------------------------------------------
// Where every output takes the same list of (key, Galois element, plaintext) -- the diagonal form of
// a layer whose packed ciphertexts share their masks -- the plaintexts go into the keys,
//   A_g[c] = sum_r sum_d D_{src(g,r),d}[sigma_r(j)] (key_{r,d}[c] pt_r)[j],
// and the rotated first polynomials as well, since ModDown divides by P and P = 0 modulo the special
// primes: A_g[0] += P sum_r sigma_r(add0_{g,r}) pt_r on the Q limbs gives the words of adding the sum after
// ModDown.  What is left is one long dot product a coefficient, reduced once.
//
// A workgroup holds 64 coefficients of one limb: the list's products in LDS (computed once for all
// outputs), a lane a coefficient, an output a wave at a time.  sigma maps aligned blocks of 64 indices
// (bit-reversed order) onto each other, so every read of D is a permuted 512-byte run.
// Primes below 2^50: words in 25-bit halves, three multiply-adds a product (the sums of x0 k0, x1 k1 and
// (x0 + x1)(k0 + k1) stay below 2^64 for 4095 terms).  Wider ones: 128-bit sums (ku_rotations).
// What bounds it: the latency of those reads (18 GB, of which a third hits L2) beside multiply-adds of
// 1.1 ms at their issue rate.  Waves that share their outputs halve the bytes past L2 but fold more sums:
// 2.7 ms and more; two outputs a wave read LDS half as often but leave twelve waves: 2.55 ms; sixteen
// waves of one output, one rotation ahead 2.29 ms, two ahead 2.26 ms (6400-node skeleton layer: 128
// outputs, 24 rotations, 4 digits, 9 limbs at N = 2^14).  Output by output with 128-bit sums the same
// products took 3.90 ms, and the first polynomials' part after ModDown 0.73 ms.
constexpr int KU_T = 1024;
struct UJob {
  const uint64_t* key;
  const uint64_t* pt;
  uint64_t g;
};
struct USrc {
  const uint64_t* add0;
  int64_t src;
};
constexpr int ku_words(int nd) { return (2 * nd + 1) * 64 + 32; }   // LDS words of one rotation

template <int ND>
__global__ __launch_bounds__(KU_T) void k_keymac_uniform(const uint64_t* __restrict__ D, const UJob* __restrict__ jobs,
                                                         const USrc* __restrict__ srcs, int R, int r0, int nr,
                                                         int n_grp, uint64_t* __restrict__ A, int accumulate, int ext,
                                                         int l1, int L, int n_mod, int log_n,
                                                         const Mod* __restrict__ mods,
                                                         const Fold25* __restrict__ folds) {
  extern __shared__ uint64_t lds[];
  uint64_t* const kx = lds;                                    // [nr][2 ND][64] keys times plaintext
  uint64_t* const px = kx + (size_t)nr * 2 * ND * 64;          // [nr][64] P times plaintext
  uint32_t* const jx = (uint32_t*)(px + (size_t)nr * 64);      // [nr][64] sigma(j)
  const size_t N = (size_t)1 << log_n;
  const int i = blockIdx.y, mi = i < l1 ? i : i - l1 + L;
  const uint32_t j0 = blockIdx.x * 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Mod m = cld(mods + mi);
  const Fold25 f = cld(folds + mi);
  const bool narrow = m.q < (1ull << 50);
  auto halves = [](uint64_t x) { return (x & M25) | (x >> 25) << 32; };
  // a wave prepares one of a rotation's 2 ND + 1 rows at a time
  for (int u = wave; u < nr * (2 * ND + 1); u += KU_T / 64) {
    const int r = u / (2 * ND + 1), e = u % (2 * ND + 1);
    const UJob jb = cld(jobs + r0 + r);
    const uint64_t p = jb.pt ? gld(jb.pt + (size_t)i * N + j0 + lane) : 1;
    if (e == 2 * ND) {
      const uint64_t v = i < l1 ? mul_mod(f.P, p, m) : 0;
      px[r * 64 + lane] = narrow ? halves(v) : v;
      jx[r * 64 + lane] = auto_idx(j0 + lane, jb.g, log_n);
    } else {
      uint64_t v = gld(jb.key + ((size_t)e * n_mod + mi) * N + j0 + lane);
      if (jb.pt) v = mul_mod(v, p, m);
      kx[(r * 2 * ND + e) * 64 + lane] = narrow ? halves(v) : v;
    }
  }
  __syncthreads();
  const IntQ iq = make_intq(m.q);
  const bool fp = fp_prime(m.q);
  const double qd = (double)m.q;
  const bool q_limb = i < l1;
  // the words of the next rotations are on their way: two ahead where the registers allow it
  constexpr int B = ND <= 4 ? 3 : 2;
  uint64_t x[B][ND], y[B];
  for (int gi = wave; gi < n_grp; gi += KU_T / 64) {
    const USrc* ss = srcs + (size_t)gi * R + r0;
    auto load = [&](uint64_t (&xx)[ND], uint64_t& yy, int r) {
      const uint32_t jj = jx[r * 64 + lane];
      const USrc s = cld(ss + r);
      const uint64_t* d = D + ((size_t)s.src * ND * ext + i) * N;
#pragma unroll
      for (int t = 0; t < ND; ++t) xx[t] = d[(size_t)t * ext * N + jj];
      yy = q_limb ? gld(s.add0 + (size_t)i * N + jj) : 0;
    };
    auto walk = [&](auto&& step) {
#pragma unroll
      for (int u = 0; u < B - 1; ++u)
        if (u < nr) load(x[u], y[u], u);
      for (int r = 0; r < nr; r += B)
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (r + u >= nr) break;
          if (r + u + B - 1 < nr) load(x[(u + B - 1) % B], y[(u + B - 1) % B], r + u + B - 1);
          step(x[u], y[u], r + u);
        }
    };
    uint64_t* out = A + ((size_t)gi * 2 * ext + i) * N + j0 + lane;
    auto put = [&](uint64_t v, int c) {
      uint64_t* o = out + (size_t)c * ext * N;
      *o = accumulate ? add_mod(v, *o, m.q) : v;
    };
    if (narrow) {
      uint64_t a[2] = {0, 0}, b[2] = {0, 0}, h[2] = {0, 0};
      auto mac = [&](uint64_t w, uint64_t k, int c) {
        const uint32_t w0 = (uint32_t)w & M25, w1 = (uint32_t)(w >> 25), k0 = (uint32_t)k, k1 = (uint32_t)(k >> 32);
        a[c] += (uint64_t)w0 * k0;
        h[c] += (uint64_t)w1 * k1;
        b[c] += (uint64_t)(w0 + w1) * (k0 + k1);
      };
      walk([&](const uint64_t (&xx)[ND], uint64_t yy, int r) {
#pragma unroll
        for (int t = 0; t < ND; ++t)
#pragma unroll
          for (int c = 0; c < 2; ++c) mac(xx[t], kx[(r * 2 * ND + 2 * t + c) * 64 + lane], c);
        mac(yy, px[r * 64 + lane], 0);
      });
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const uint64_t mid = b[c] - a[c] - h[c];
        put(fp ? fold25_fp(a[c], mid, h[c], qd, m.qinv, f) : fold25_int(a[c], mid, h[c], m.q, iq, f), c);
      }
    } else {
      u128 s0 = 0, s1 = 0;
      walk([&](const uint64_t (&xx)[ND], uint64_t yy, int r) {
#pragma unroll
        for (int t = 0; t < ND; ++t) {
          s0 += (u128)xx[t] * kx[(r * 2 * ND + 2 * t) * 64 + lane];
          s1 += (u128)xx[t] * kx[(r * 2 * ND + 2 * t + 1) * 64 + lane];
        }
        if (q_limb) s0 += (u128)yy * px[r * 64 + lane];
      });
      put(reduce128(s0, m), 0);
      put(reduce128(s1, m), 1);
    }
  }
}

// The masked key inner products of a chunk with its jobs taken key by key (runs of jobs
// sharing one key and Galois element, at most KM_MAXG output groups): a thread per (coefficient,
// limb) reads each key word once for its run and adds every job's product, times its
// plaintext, to its group's sum.  The runs are split in n_seg segments (blockIdx.z) whose sums
// go to P[seg][group][component] and are added to the accumulators by k_masked_combine.
// Limbs of Q primes in (2^49, 2^50) (fq): the products in fp64 residues (fpmod.h), each an
// exact signed representative in (-q, q); a job's digit sum is brought back before its mask
// product, and the group sums every four jobs, so every double stays an exact integer below
// 2^53.  The words equal those of the integer form, which the special primes' limbs take.
constexpr int KM_MAXG = 4;
template <int ND, int NG>
__global__ void k_keymac_masked_runs(const uint64_t* __restrict__ D, const KSJob* __restrict__ jobs,
                                     const int* __restrict__ run_start, int n_runs, int n_seg,
                                     const int* __restrict__ job_gl, int n_gl, uint64_t* __restrict__ P, int ext,
                                     int l1, int L, int n_mod, int log_n, int fq, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const uint32_t j = blockIdx.x * KB + threadIdx.x;
  const int i = blockIdx.y, seg = blockIdx.z;
  const int m = i < l1 ? i : i - l1 + L;
  const Mod md = mods[m];
  const int ra = (int)((int64_t)n_runs * seg / n_seg), rb = (int)((int64_t)n_runs * (seg + 1) / n_seg);
  if (fq && i < l1) {
    const double qd = (double)md.q, qinv = md.qinv;
    auto cv = [](uint64_t v) { return b2f(to_fbits(v)); };
    double T0[NG], T1[NG];
    int cnt[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      T0[g] = T1[g] = 0.0;
      cnt[g] = 0;
    }
    for (int run = ra; run < rb; ++run) {
      const int r0 = run_start[run], r1 = run_start[run + 1];
      const KSJob j0 = jobs[r0];
      const uint32_t jj = j0.g == 1 ? j : auto_idx(j, j0.g, log_n);
      double k0[ND], k1[ND];
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        k0[d] = cv(gld(j0.key + (((size_t)d * 2 + 0) * n_mod + m) * N + j));
        k1[d] = cv(gld(j0.key + (((size_t)d * 2 + 1) * n_mod + m) * N + j));
      }
      for (int r = r0; r < r1; ++r) {
        const KSJob jb = jobs[r];
        const uint64_t* Du = D + (size_t)jb.src * ND * ext * N;
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int d = 0; d < ND; ++d) {
          const double x = cv(Du[((size_t)d * ext + i) * N + jj]);
          s0 += fmulmod_s(x, k0[d], qd, qinv);
          s1 += fmulmod_s(x, k1[d], qd, qinv);
        }
        s0 = sred(s0, qd, qinv);
        s1 = sred(s1, qd, qinv);
        if (jb.pt) {   // one job per thread block step: no divergence
          const double p = cv(gld(jb.pt + (size_t)i * N + j));
          s0 = fmulmod_s(s0, p, qd, qinv);
          s1 = fmulmod_s(s1, p, qd, qinv);
        }
        const int gl = job_gl[r];
#pragma unroll
        for (int g = 0; g < NG; ++g)
          if (g == gl) {
            T0[g] += s0;
            T1[g] += s1;
            if (++cnt[g] == 4) {
              T0[g] = sred(T0[g], qd, qinv);
              T1[g] = sred(T1[g], qd, qinv);
              cnt[g] = 0;
            }
          }
      }
    }
#pragma unroll
    for (int g = 0; g < NG; ++g)
      if (g < n_gl) {
        P[((((size_t)seg * n_gl + g) * 2 + 0) * ext + i) * N + j] = from_fbits(f2b(canon(sred(T0[g], qd, qinv), qd)));
        P[((((size_t)seg * n_gl + g) * 2 + 1) * ext + i) * N + j] = from_fbits(f2b(canon(sred(T1[g], qd, qinv), qd)));
      }
    return;
  }
  u128 t0[NG], t1[NG];
  uint64_t v0[NG], v1[NG];
  int cnt[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    t0[g] = t1[g] = 0;
    v0[g] = v1[g] = 0;
    cnt[g] = 0;
  }
  for (int run = ra; run < rb; ++run) {
    const int r0 = run_start[run], r1 = run_start[run + 1];
    const KSJob j0 = jobs[r0];
    const uint32_t jj = j0.g == 1 ? j : auto_idx(j, j0.g, log_n);
    uint64_t k0[ND], k1[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      k0[d] = gld(j0.key + (((size_t)d * 2 + 0) * n_mod + m) * N + j);
      k1[d] = gld(j0.key + (((size_t)d * 2 + 1) * n_mod + m) * N + j);
    }
    for (int r = r0; r < r1; ++r) {
      const KSJob jb = jobs[r];
      const uint64_t* Du = D + (size_t)jb.src * ND * ext * N;
      u128 s0 = 0, s1 = 0;
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        const u128 x = Du[((size_t)d * ext + i) * N + jj];
        s0 += x * k0[d];
        s1 += x * k1[d];
      }
      const uint64_t x0 = reduce128(s0, md), x1 = reduce128(s1, md);
      u128 y0 = x0, y1 = x1;
      if (jb.pt) {   // one job per thread block step: no divergence
        const uint64_t p = gld(jb.pt + (size_t)i * N + j);
        y0 = (u128)x0 * p;
        y1 = (u128)x1 * p;
      }
      const int gl = job_gl[r];
#pragma unroll
      for (int g = 0; g < NG; ++g)
        if (g == gl) {
          t0[g] += y0;
          t1[g] += y1;
          if (++cnt[g] == 8) {
            v0[g] = add_mod(v0[g], reduce128(t0[g], md), md.q);
            v1[g] = add_mod(v1[g], reduce128(t1[g], md), md.q);
            t0[g] = t1[g] = 0;
            cnt[g] = 0;
          }
        }
    }
  }
#pragma unroll
  for (int g = 0; g < NG; ++g)
    if (g < n_gl) {
      P[((((size_t)seg * n_gl + g) * 2 + 0) * ext + i) * N + j] = add_mod(v0[g], reduce128(t0[g], md), md.q);
      P[((((size_t)seg * n_gl + g) * 2 + 1) * ext + i) * N + j] = add_mod(v1[g], reduce128(t1[g], md), md.q);
    }
}

// A_group += sum over the segments of P[seg][group] (both components, every limb of the key basis)
__global__ void k_masked_combine(const GroupDesc* __restrict__ groups, const uint64_t* __restrict__ P, int n_gl,
                                 int n_seg, int ext, int l1, int L, int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const uint32_t j = blockIdx.x * KB + threadIdx.x;
  const int i = blockIdx.y, g = blockIdx.z >> 1, comp = blockIdx.z & 1;
  const int m = i < l1 ? i : i - l1 + L;
  const uint64_t q = mods[m].q;
  uint64_t* a = groups[g].out + ((size_t)comp * ext + i) * N + j;
  uint64_t v = gld(a);
  for (int sg = 0; sg < n_seg; ++sg) v = add_mod(v, P[((((size_t)sg * n_gl + g) * 2 + comp) * ext + i) * N + j], q);
  gst(a, v);
}

// out_grp (+)= (A_Q - conv) P^-1  [+ sum_r sigma_g(add0_r) (.) pt_r on component 0]
__global__ void k_masked_final(const uint64_t* __restrict__ A, const uint64_t* __restrict__ conv, int ext, int l1,
                               MDK k, const KSJob* __restrict__ jobs, const MaskGroup* __restrict__ groups,
                               uint64_t* const* __restrict__ outs, int accumulate, int log_n,
                               const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const uint32_t j = blockIdx.x * KB + threadIdx.x;
  const int i = blockIdx.y;
  const int comp = blockIdx.z & 1, g = blockIdx.z >> 1;
  const Mod md = mods[i];
  const uint64_t q = md.q;
  const size_t o = ((size_t)comp * l1 + i) * N + j;
  uint64_t v = sub_mod(A[(((size_t)g * 2 + comp) * ext + i) * N + j], conv[(((size_t)g * 2 + comp) * l1 + i) * N + j], q);
  v = mul_shoup(v, k.pinv[i], k.pinv_s[i], q);
  if (comp == 0) {
    const MaskGroup gr = groups[g];
    u128 s = 0;
    int cnt = 0;
    for (int r = gr.start; r < gr.end; ++r) {
      const KSJob jb = jobs[r];
      if (!jb.add0) continue;
      const uint64_t x = gld(jb.add0 + (size_t)i * N + (jb.g == 1 ? j : auto_idx(j, jb.g, log_n)));
      s += jb.pt ? (u128)x * gld(jb.pt + (size_t)i * N + j) : (u128)x;
      if (++cnt == 8) {
        v = add_mod(v, reduce128(s, md), q);
        s = 0;
        cnt = 0;
      }
    }
    v = add_mod(v, reduce128(s, md), q);
  }
  uint64_t* out = outs[g];
  gst(out + o, accumulate ? add_mod(gld(out + o), v, q) : v);
}

enum { S_KM_A = 80, S_KM_CONV, S_KM_JOBS, S_KM_OUT, S_KM_P };

// rotations a launch takes: its LDS, and the sums' room (narrow words: 4095 products of 2^52; wide
// ones: products of two words below 2^bits in 128 bits)
static int ku_rotations(ckks_ctx* c, int nd) {
  const int bits = std::max(c->q_bits, c->p_bits);
  const int wide = 2 * bits >= 128 ? 1 : 1 << std::min(12, 128 - 2 * bits);
  const int most = std::min((144 << 10) / (ku_words(nd) * 8), std::min(4095, wide - 1) / (nd + 1));
  return most;
}

// The sources of the output that has the most, where every output's list of (key, Galois element,
// plaintext) is the first one's and has its add0s; 0 where it is not
static size_t uniform_jobs(const std::vector<KSJob>& jobs, int n_grp, size_t n_sources) {
  if (n_grp < 1 || jobs.empty() || jobs.size() % n_grp) return 0;
  const size_t R = jobs.size() / n_grp;
  std::vector<int> seen(n_sources, -1);   // the last output that read a source
  size_t most = 0, n = 0;
  for (size_t k = 0; k < jobs.size(); ++k) {
    const KSJob &a = jobs[k], &b = jobs[k % R];
    if (a.grp != (int)(k / R) || a.key != b.key || a.g != b.g || a.pt != b.pt || !a.add0) return 0;
    if (k % R == 0) n = 0;
    if (seen[a.src] != a.grp) ++n;
    seen[a.src] = a.grp;
    most = std::max(most, n);
  }
  return most;
}

// Whether the sums of n_grp outputs with n_src sources each are faster with the list's products shared
// (k_keymac_uniform) than output by output (k_keymac_masked).  Making the products takes nd ext N / 64 rounds of
// 2 nd + 1 words a rotation, whatever the number of outputs, and a workgroup's sixteen waves take an output each: so
// where there are many rounds it needs outputs to share them, and where there are few the launch is short either
// way and the saved passes count.  Both sides with ModUp and ModDown (us; shared, by output), rotations from one source:
//   N = 2^14, 7 limbs, 49 rotations: 5 outputs 783, 577; 10 955, 918; 12 992, 1044; 16 1081, 1320; 48 2316, 3723
//   N = 2^16, 7 limbs, 49: 5 outputs 3020, 1804; 8 3302, 2735; 16 4082, 5148
//   N = 2^13, 16 limbs, 48: 5 outputs 1265, 858; 12 1588, 1627
//   2304 rounds (N = 2^12, 7 limbs, 25): 5 outputs 183, 181; 8 197, 205; 1536 rounds (N = 2^13, 3 limbs, 48):
//   5 outputs 208, 228; 3072 rounds (N = 2^14, 3 limbs, 49): 5 outputs 340, 281; 10 416, 411; 12 440, 474
// Where every rotation has a source of its own (giant steps) each wave reads its output's digits alone, from all
// over memory: N = 2^14, 7 limbs, 114 of them: 5 outputs 4739, 3770; 16 16168, 12257; 32 30449, 23885; N = 2^13,
// 7 limbs, 77: 16 outputs 4396, 4077.  A ring of 2^12 has its digits in cache: 16 limbs, 7 of them: 16 outputs 744,
// 772; N = 2^11, 3 limbs, 24: 5 outputs 136, 170.
static bool uniform_pays(const ckks_ctx* c, int nd, int ext, int n_grp, size_t n_src) {
  const size_t rounds = (size_t)nd * ext * c->N / 64;
  return (n_src == 1 || c->log_n <= 12) && (rounds <= 2304 || n_grp >= 12);
}

// The masked sums of outputs that share their list: A [n_grp][2][ext][N], first polynomials included
static void masked_uniform(ckks_ctx* c, int level, const std::vector<const uint64_t*>& sources,
                           const std::vector<KSJob>& jobs, int n_grp, uint64_t* A) {
  const size_t N = c->N;
  const int l1 = level + 1, ext = l1 + c->alpha;
  const int nd = (l1 + c->alpha - 1) / c->alpha;
  const int R = (int)(jobs.size() / n_grp);
  const size_t per_src = (size_t)(nd * ext + l1) * N * 8;
  std::vector<UJob> list;
  for (int r = 0; r < R; ++r) list.push_back(UJob{jobs[r].key, jobs[r].pt, jobs[r].g});
  for (int ga = 0; ga < n_grp;) {
    // whole outputs, as many as their sources' digits allow
    std::vector<int> local(sources.size(), -1);
    std::vector<const uint64_t*> srcs;
    std::vector<USrc> us;
    int gb = ga;
    for (; gb < n_grp; ++gb) {
      size_t fresh = 0;
      std::vector<char> seen(sources.size(), 0);
      for (int r = 0; r < R; ++r) {
        const int s = jobs[(size_t)gb * R + r].src;
        if (local[s] < 0 && !seen[s]) ++fresh;
        seen[s] = 1;
      }
      if (gb > ga && (srcs.size() + fresh) * per_src > KS_BUDGET) break;
      for (int r = 0; r < R; ++r) {
        const KSJob& jb = jobs[(size_t)gb * R + r];
        if (local[jb.src] < 0) {
          local[jb.src] = (int)srcs.size();
          srcs.push_back(sources[jb.src]);
        }
        us.push_back(USrc{jb.add0, local[jb.src]});
      }
    }
    const int U = (int)srcs.size(), ng = gb - ga;
    const auto [jd, ud, sd] = upload(c, S_KB_JOBS, list, us, srcs);
    uint64_t* tmp = (uint64_t*)dev_scratch(c, S_KB_TMP, (size_t)U * l1 * N * 8);
    uint64_t* D = (uint64_t*)dev_scratch(c, S_KB_D, (size_t)U * nd * ext * N * 8);
    {
      ProfScope pm(c, "modup");
      modup_batch(c, level, sd, U, tmp, D);
    }
    {
      ProfScope pk(c, "keymac");
      const int most = ku_rotations(c, nd);
      for (int r0 = 0; r0 < R; r0 += most) {
        const int nr = std::min(most, R - r0);
        uint64_t* Ag = A + (size_t)ga * 2 * ext * N;
        const size_t bytes = (size_t)nr * ku_words(nd) * 8;
#define KU_LAUNCH(NDV)                                                                                                \
  hipLaunchKernelGGL(k_keymac_uniform<NDV>, dim3(N / 64, ext), dim3(KU_T), bytes, c->stream, D, jd, ud, R, r0, nr, ng, \
                     Ag, r0 ? 1 : 0, ext, l1, c->L, c->n_mod(), c->log_n, c->t.mods, c->t.fold25)
        switch (nd) {
          case 1: KU_LAUNCH(1); break;
          case 2: KU_LAUNCH(2); break;
          case 3: KU_LAUNCH(3); break;
          case 4: KU_LAUNCH(4); break;
          case 5: KU_LAUNCH(5); break;
          case 6: KU_LAUNCH(6); break;
          case 7: KU_LAUNCH(7); break;
          default: KU_LAUNCH(8);
        }
#undef KU_LAUNCH
        HIPCHECK(hipGetLastError());
      }
    }
    ga = gb;
  }
}

void keyswitch_masked_sum(ckks_ctx* c, int level, const std::vector<const uint64_t*>& sources,
                          const std::vector<KSJob>& jobs, const std::vector<uint64_t*>& outs, bool accumulate) {
  const size_t N = c->N;
  const int l1 = level + 1, ext = l1 + c->alpha;
  const int nd = (l1 + c->alpha - 1) / c->alpha;
  const int n_grp = (int)outs.size();
  if (c->alpha > 8 || l1 > 64 || nd > DigitTables::MAX) FICGCN_THROW(EINVAL_, "too many primes");
  if (n_grp == 0) return;
  for (size_t r = 0; r < jobs.size(); ++r) {
    const KSJob& jb = jobs[r];
    if (jb.src < 0 || jb.src >= (int)sources.size() || !sources[jb.src] || !jb.key || jb.grp < 0 ||
        jb.grp >= n_grp || (r && jobs[r - 1].grp > jb.grp))
      FICGCN_THROW(EINVAL_, "bad masked key-switch job");
  }
  for (uint64_t* o : outs)
    if (!o) FICGCN_THROW(EINVAL_, "null output");
  // at most KM_MAXG outputs: the jobs go key by key (before chunking, so a chunk holds every use
  // of its keys) and every key is read once for all outputs that use it
  const bool by_key = n_grp <= KM_MAXG && nd <= KR_MAXD;
  std::vector<KSJob> sorted_jobs;
  if (by_key) {
    sorted_jobs = jobs;
    std::stable_sort(sorted_jobs.begin(), sorted_jobs.end(), [](const KSJob& x, const KSJob& y) {
      return x.key != y.key ? x.key < y.key : x.g < y.g;
    });
  }
  const std::vector<KSJob>& jl = by_key ? sorted_jobs : jobs;
  ProfScope ps(c, "ks_masked");
  // one accumulator on the key basis per output, summed over every chunk
  uint64_t* A = (uint64_t*)dev_scratch(c, S_KM_A, (size_t)n_grp * 2 * ext * N * 8);
  const size_t per_src = (size_t)(nd * ext + l1) * N * 8;
  // an output's sources lie in one chunk there, so they have to fit it (giant steps bring one a rotation: 140
  // of them at N = 2^16 and 16 limbs are 11.7 GB)
  const size_t n_src = fused_basis(c) && !by_key && nd <= KR_MAXD ? uniform_jobs(jobs, n_grp, sources.size()) : 0;
  if (n_src && uniform_pays(c, nd, ext, n_grp, n_src) && (n_src == 1 || n_src * per_src <= KS_BUDGET)) {
    masked_uniform(c, level, sources, jobs, n_grp, A);
    std::vector<FinalJob> finals;
    for (uint64_t* o : outs) finals.push_back(FinalJob{o, nullptr, nullptr, 1, accumulate ? 1 : 0, 0});
    const auto [fd] = upload(c, S_KM_OUT, finals);
    uint64_t* conv = (uint64_t*)dev_scratch(c, S_KM_CONV, (size_t)n_grp * 2 * l1 * N * 8);
    ProfScope pd(c, "moddown");
    moddown_polys(c, level, A, 2 * n_grp, conv, false);
    moddown_final(c, level, A, conv, fd, FinalJob{}, n_grp);
    return;
  }
  zero_fill(c, A, (size_t)n_grp * 2 * ext * N);
  const size_t per_job = 0;   // a job's products go straight into its output's accumulator
  size_t a = 0;
  while (a < jl.size()) {
    std::vector<int> local(sources.size(), -1);
    std::vector<const uint64_t*> srcs;
    std::vector<KSJob> cj;
    size_t b = a, bytes = 0;
    while (b < jl.size()) {
      const bool new_src = local[jl[b].src] < 0;
      const size_t add = per_job + (new_src ? per_src : 0);
      // a chunk ends between runs of one key when the jobs go key by key
      const bool run_start = !by_key || b == a || jl[b].key != jl[b - 1].key || jl[b].g != jl[b - 1].g;
      if (b > a && run_start && bytes + add > KS_BUDGET) break;
      bytes += add;
      if (new_src) {
        local[jl[b].src] = (int)srcs.size();
        srcs.push_back(sources[jl[b].src]);
      }
      KSJob jc = jl[b];
      jc.src = local[jc.src];
      cj.push_back(jc);
      ++b;
    }
    // this chunk's job ranges per output, each pointing at the output's accumulator
    std::vector<GroupDesc> gds;
    if (by_key) {
      for (int g = 0; g < n_grp; ++g) gds.push_back(GroupDesc{A + (size_t)g * 2 * ext * N, 0, 0, 1, 0});
    } else {
      for (size_t r = 0; r < cj.size(); ++r) {
        const int g = cj[r].grp;
        if (r == 0 || cj[r - 1].grp != g)
          gds.push_back(GroupDesc{A + (size_t)g * 2 * ext * N, (int)r, (int)r + 1, 1, 0});
        else
          gds.back().end = (int)r + 1;
      }
    }
    const int U = (int)srcs.size();
    // by key: runs of jobs that share one, and each job's output
    std::vector<int> runs, kgl;
    if (by_key) {
      runs = key_runs(cj);
      for (const KSJob& jb : cj) kgl.push_back(jb.grp);
    }
    const auto [jd, sd, gd, rd, gld_] = upload(c, S_KB_JOBS, cj, srcs, gds, runs, kgl);
    uint64_t* tmp = (uint64_t*)dev_scratch(c, S_KB_TMP, (size_t)U * l1 * N * 8);
    uint64_t* D = (uint64_t*)dev_scratch(c, S_KB_D, (size_t)U * nd * ext * N * 8);
    {
      ProfScope pm(c, "modup");
      modup_batch(c, level, sd, U, tmp, D);
    }
    {
      ProfScope pk(c, "keymac");
      if (gds.size() > 65535) FICGCN_THROW(EINVAL_, "too many outputs in one launch");
      const int n_jb = (int)(N / KB), ng = (int)gds.size();
      if (by_key) {
        // each key read once for every output that uses it; runs split in segments for parallelism
        const int n_runs = (int)runs.size() - 1;
        const int n_seg = std::max(1, std::min(32, n_runs / 8));
        uint64_t* P = (uint64_t*)dev_scratch(c, S_KM_P, (size_t)n_seg * ng * 2 * ext * N * 8);
        const dim3 grid(n_jb, ext, n_seg);
        int fq = 1;   // the Q limbs in fp64 residues when every Q prime of the level lies in (2^49, 2^50)
        for (int qi = 0; qi < l1; ++qi) fq = fq && c->mod[qi] > (1ull << 49) && c->mod[qi] < (1ull << 50);
#define KM_LAUNCH(NDV, NGV)                                                                                \
  hipLaunchKernelGGL((k_keymac_masked_runs<NDV, NGV>), grid, dim3(KB), 0, c->stream, D, jd, rd, n_runs, n_seg, gld_, \
                     ng, P, ext, l1, c->L, c->n_mod(), c->log_n, fq, c->t.mods)
#define KM_BY_G(NDV)             \
  switch (ng) {                  \
    case 1: KM_LAUNCH(NDV, 1); break; \
    case 2: KM_LAUNCH(NDV, 2); break; \
    case 3: KM_LAUNCH(NDV, 3); break; \
    default: KM_LAUNCH(NDV, 4);  \
  }
        switch (nd) {
          case 1: KM_BY_G(1); break;
          case 2: KM_BY_G(2); break;
          case 3: KM_BY_G(3); break;
          case 4: KM_BY_G(4); break;
          case 5: KM_BY_G(5); break;
          case 6: KM_BY_G(6); break;
          case 7: KM_BY_G(7); break;
          default: KM_BY_G(8);
        }
#undef KM_BY_G
#undef KM_LAUNCH
        HIPCHECK(hipGetLastError());
        hipLaunchKernelGGL(k_masked_combine, dim3(n_jb, ext, 2 * ng), dim3(KB), 0, c->stream, gd, P, ng, n_seg, ext,
                           l1, c->L, c->log_n, c->t.mods);
      } else {
        const bool xcd = n_jb % 8 == 0 && (size_t)n_jb * ng < ((size_t)1 << 31);
        const dim3 grid = xcd ? dim3(n_jb * ng, ext, 1) : dim3(n_jb, ext, ng);
        hipLaunchKernelGGL(k_keymac_masked, grid, dim3(KB), 0, c->stream, D, jd, gd, nd, ext, l1, c->L, c->n_mod(),
                           c->log_n, ng, xcd ? 1 : 0, c->t.mods);
      }
      HIPCHECK(hipGetLastError());
    }
    a = b;
  }
  // one ModDown per output: P limbs to coefficient form, rounded conversion,
  // forward NTT, then out (+)= (A_Q - conv) P^-1 + sum sigma(add0) (.) pt
  {
    ProfScope pd(c, "moddown");
    const MDK& k = c->mdk[level];
    std::vector<MaskGroup> mg(n_grp, MaskGroup{0, 0});
    for (size_t r = 0; r < jobs.size(); ++r) {
      const int g = jobs[r].grp;
      if (mg[g].end == 0) mg[g].start = (int)r;
      mg[g].end = (int)r + 1;
    }
    const auto [jall, mgd, od] = upload(c, S_KM_JOBS, jobs, mg, outs);
    uint64_t* conv = (uint64_t*)dev_scratch(c, S_KM_CONV, (size_t)n_grp * 2 * l1 * N * 8);
    moddown_conv_batch(c, level, A, 2 * n_grp, k, conv);
    hipLaunchKernelGGL(k_masked_final, dim3(N / KB, l1, 2 * n_grp), dim3(KB), 0, c->stream, A, conv, ext, l1, k, jall,
                       mgd, od, accumulate ? 1 : 0, c->log_n, c->t.mods);
    HIPCHECK(hipGetLastError());
  }
}

// ---- batched ciphertext kernels --------------------------------------------------

// d = (x0 y0, x0 y1 + x1 y0, x1 y1) per job, [3][l1][N]
__global__ void k_tensor_batch(const TensorJob* __restrict__ jobs, int l1, int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const size_t j = blockIdx.x * (size_t)KB + threadIdx.x;
  const int i = blockIdx.y;
  const TensorJob jb = jobs[blockIdx.z];
  const Mod m = mods[i];
  const size_t o0 = i * N + j, o1 = (l1 + i) * N + j;
  const uint64_t x0 = gld(jb.x + o0), x1 = gld(jb.x + o1), y0 = gld(jb.y + o0), y1 = gld(jb.y + o1);
  gst(jb.d + o0, reduce128((u128)x0 * y0, m));
  gst(jb.d + o1, reduce128((u128)x0 * y1 + (u128)x1 * y0, m));
  gst(jb.d + (2 * l1 + i) * N + j, reduce128((u128)x1 * y1, m));
}

void tensor_batch(ckks_ctx* c, int level, const std::vector<TensorJob>& jobs) {
  if (jobs.empty()) return;
  const auto [jd] = upload(c, S_TB_JOBS, jobs);
  hipLaunchKernelGGL(k_tensor_batch, dim3(c->N / KB, level + 1, jobs.size()), dim3(KB), 0, c->stream, jd, level + 1,
                     c->log_n, c->t.mods);
  HIPCHECK(hipGetLastError());
}

// c'_i = (c_i + d_i) q_l^-1, compacted in place from [2][l+1][N] to [2][l][N].
// One thread walks the limbs of one component upwards, so a limb is read
// before the write of the next-lower position reaches it; the two
// components write disjoint ranges.
__global__ void k_rs_final(uint64_t* const* __restrict__ cts, const uint64_t* __restrict__ d, int lvl, RSK k, int log_n,
                           const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const size_t j = blockIdx.x * (size_t)KB + threadIdx.x;
  const int z = blockIdx.y;
  const int comp = z & 1;
  uint64_t* ct = cts[z >> 1];
  for (int i = 0; i < lvl; ++i) {
    const uint64_t q = mods[i].q;
    const uint64_t v = add_mod(gld(ct + ((size_t)comp * (lvl + 1) + i) * N + j), d[((size_t)z * lvl + i) * N + j], q);
    gst(ct + ((size_t)comp * lvl + i) * N + j, mul_shoup(v, k.inv[i], k.inv_s[i], q));
  }
}

void rescale_batch(ckks_ctx* c, int level, const std::vector<uint64_t*>& cts) {
  if (cts.empty()) return;
  if (level < 1) FICGCN_THROW(ELEVEL_, "rescale at level 0");
  if (level > 63) FICGCN_THROW(EINVAL_, "too many primes");
  ProfScope ps(c, "rescale");
  const size_t N = c->N;
  const int n = (int)cts.size();
  const auto [cd] = upload(c, S_RS_PTR, cts);
  uint64_t* last = (uint64_t*)dev_scratch(c, S_RS_LAST, (size_t)2 * n * N * 8);
  uint64_t* d = (uint64_t*)dev_scratch(c, S_RS_D, (size_t)2 * n * level * N * 8);
  const RSK& k = c->rsk[level];
  rescale_prep(c, level, cd, nullptr, n, last, d);
  hipLaunchKernelGGL(k_rs_final, dim3(N / KB, 2 * n), dim3(KB), 0, c->stream, cd, d, level, k, c->log_n, c->t.mods);
  HIPCHECK(hipGetLastError());
}

// Two rescales in one call, c'' = round(round(c / q_l) / q_{l-1}), word for
// word.  With x_l and x_{l-1} the last two limbs in coefficient form,
//   d_i = (h_l - [x_l + h_l]_{q_l}) mod q_i            (first correction),
//   y   = (x_{l-1} + d_{l-1}) q_l^-1 mod q_{l-1}        (limb l-1 after it),
//   e_i = (h_{l-1} - [y + h_{l-1}]_{q_{l-1}}) mod q_i   (second correction),
// and, the NTT being linear modulo each q_i, for i < l - 1
//   c''_i = c_i (q_l q_{l-1})^-1 + NTT_i((d_i q_l^-1 + e_i) q_{l-1}^-1)  mod q_i,
// which is what two rescales in a row compute, with one forward NTT of l - 1
// limbs instead of l + (l - 1).  h_k = floor(q_k / 2).
constexpr int RS2_MAX = 32;
struct RSK2 {
  uint64_t inv12[RS2_MAX], inv12_s[RS2_MAX];    // (q_l q_{l-1})^-1 mod q_i, Shoup
};

// c''_i = c_i (q_l q_{l-1})^-1 + f_i, compacted in place from [2][l+1][N] to
// [2][l-1][N]: one thread walks the limbs of one component upwards, so each
// write lands on a limb this thread has already read (or on a dropped limb of
// the first component, which no thread reads).
__global__ void k_rs2_final(uint64_t* const* __restrict__ cts, const uint64_t* __restrict__ f, int lvl, RSK2 k,
                            int log_n, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  const size_t j = blockIdx.x * (size_t)KB + threadIdx.x;
  const int z = blockIdx.y;
  const int comp = z & 1;
  uint64_t* ct = cts[z >> 1];
  for (int i = 0; i < lvl - 1; ++i) {
    const uint64_t q = mods[i].q;
    const uint64_t v = mul_shoup(gld(ct + ((size_t)comp * (lvl + 1) + i) * N + j), k.inv12[i], k.inv12_s[i], q);
    gst(ct + ((size_t)comp * (lvl - 1) + i) * N + j, add_mod(v, f[((size_t)z * (lvl - 1) + i) * N + j], q));
  }
}

void rescale2_batch(ckks_ctx* c, int level, const std::vector<uint64_t*>& cts) {
  if (cts.empty()) return;
  if (level < 2 || level > RS2_MAX) {
    rescale_batch(c, level, cts);
    rescale_batch(c, level - 1, cts);
    return;
  }
  ProfScope ps(c, "rescale");
  const size_t N = c->N;
  const int n = (int)cts.size();
  const auto [cd] = upload(c, S_RS_PTR, cts);
  uint64_t* last = (uint64_t*)dev_scratch(c, S_RS_LAST, (size_t)2 * n * 2 * N * 8);
  uint64_t* f = (uint64_t*)dev_scratch(c, S_RS_D, (size_t)2 * n * (level - 1) * N * 8);
  RSK2 k{};
  const RSK &r1 = c->rsk[level], &r2 = c->rsk[level - 1];
  for (int i = 0; i < level - 1; ++i) {
    const uint64_t q = c->mod[i];
    k.inv12[i] = (uint64_t)((u128)r1.inv[i] * r2.inv[i] % q);
    k.inv12_s[i] = shoup(k.inv12[i], q);
  }
  rescale2_prep(c, level, cd, n, last, f);
  hipLaunchKernelGGL(k_rs2_final, dim3(N / KB, 2 * n), dim3(KB), 0, c->stream, cd, f, level, k, c->log_n, c->t.mods);
  HIPCHECK(hipGetLastError());
}

// outs[g] (+)= sum over the terms of group g of ct (.) pt, or ct when pt is null
__global__ void k_group_mac(const MacTerm* __restrict__ terms, const int* __restrict__ group_start,
                            uint64_t* const* __restrict__ outs, int l1, int accumulate, int log_n, int n_groups,
                            int xcd_order, const Mod* __restrict__ mods) {
  const size_t N = (size_t)1 << log_n;
  // limb slowest: one limb of every group's terms is in flight at a time.
  // With xcd_order, blocks go round-robin over the 8 XCDs by linear id, so
  // block b runs coefficient block 8 (b / 8 / n_groups) + b % 8 for group
  // (b / 8) % n_groups: every group of one coefficient block runs on one XCD,
  // back to back, and the ciphertexts the groups share (baby steps) are read
  // into that XCD's L2 once.  One thread takes both components of a
  // coefficient: each plaintext word is read once for the two products.
  const int i = blockIdx.z;
  int jb, g;
  if (xcd_order) {
    const int b = blockIdx.x, idx = b >> 3;
    jb = (b & 7) + 8 * (idx / n_groups);
    g = idx % n_groups;
  } else {
    jb = blockIdx.x;
    g = blockIdx.y;
  }
  const size_t j = (size_t)jb * KB + threadIdx.x;
  const Mod m = mods[i];
  const size_t o0 = (size_t)i * N + j, o1 = ((size_t)l1 + i) * N + j;
  uint64_t* out = outs[g];
  uint64_t a0 = accumulate ? gld(out + o0) : 0, a1 = accumulate ? gld(out + o1) : 0;
  // A term without a plaintext adds its ciphertext: it is multiplied by a
  // stored 1 instead (the words are below q, so the sum is the same), which
  // keeps the term loop free of branches.  Terms go in fours: the twelve loads
  // of four terms are issued before their products, summed in 128 bits and
  // reduced once per four.
  const size_t pj = (size_t)i * N + j;
  auto load = [&](int t, uint64_t& x0, uint64_t& x1, uint64_t& p) {
    const MacTerm tm = terms[t];
    x0 = gld(tm.ct + (tm.l1 ? pj : o0));
    x1 = gld(tm.ct + (tm.l1 ? ((size_t)tm.l1 + i) * N + j : o1));
    p = gld(tm.pt ? tm.pt + pj : &k_one_word);
  };
  const int t_end = group_start[g + 1];
  int t = group_start[g];
  for (; t + 4 <= t_end; t += 4) {
    uint64_t x0[4], x1[4], p[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) load(t + u, x0[u], x1[u], p[u]);
    u128 s0 = 0, s1 = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      s0 += (u128)x0[u] * p[u];
      s1 += (u128)x1[u] * p[u];
    }
    a0 = add_mod(a0, reduce128(s0, m), m.q);
    a1 = add_mod(a1, reduce128(s1, m), m.q);
  }
  u128 s0 = 0, s1 = 0;
  for (; t < t_end; ++t) {
    uint64_t x0, x1, p;
    load(t, x0, x1, p);
    s0 += (u128)x0 * p;
    s1 += (u128)x1 * p;
  }
  gst(out + o0, add_mod(a0, reduce128(s0, m), m.q));
  gst(out + o1, add_mod(a1, reduce128(s1, m), m.q));
}

void group_mac(ckks_ctx* c, int level, const std::vector<std::vector<MacTerm>>& groups,
               const std::vector<uint64_t*>& outs, bool accumulate) {
  if (groups.empty()) return;
  if (groups.size() != outs.size()) FICGCN_THROW(EINVAL_, "group/output count mismatch");
  ProfScope ps(c, "group_mac");
  std::vector<MacTerm> flat;
  std::vector<int> start{0};
  for (const auto& g : groups) {
    for (const MacTerm& t : g)
      if (!t.ct) FICGCN_THROW(EINVAL_, "null term");
    flat.insert(flat.end(), g.begin(), g.end());
    start.push_back((int)flat.size());
  }
  for (uint64_t* o : outs)
    if (!o) FICGCN_THROW(EINVAL_, "null output");
  const auto [td, sd, od] = upload(c, S_GM_TERMS, flat, start, outs);
  if (groups.size() > 65535) FICGCN_THROW(EINVAL_, "too many groups in one launch");
  const int n_jb = c->N / KB, ng = (int)groups.size();
  const bool xcd = n_jb % 8 == 0 && (size_t)n_jb * ng < ((size_t)1 << 31);
  const dim3 grid = xcd ? dim3(n_jb * ng, 1, level + 1) : dim3(n_jb, ng, level + 1);
  hipLaunchKernelGGL(k_group_mac, grid, dim3(KB), 0, c->stream, td, sd, od, level + 1, accumulate ? 1 : 0, c->log_n, ng,
                     xcd ? 1 : 0, c->t.mods);
  HIPCHECK(hipGetLastError());
}


// ---- masked sums of several ciphertexts under shared masks ----------------------

// outs[g * NP + c] (+)= sum over the terms of group g of ct_c (.) pt (ct_c alone when pt is
// null).  The NP ciphertexts of a term share its plaintext word, read once; a thread takes
// two neighbouring coefficients of one limb with 16-byte loads, so every load instruction
// moves two words and NP + 1 streams are in flight per term.
// GM_TB threads per block: the baby-step ciphertexts of one block's 2 GM_TB coefficients
// (every packed ciphertext, both components) stay in L2 while the masks stream past them.
//
// Products, by the level's primes: all in (2^49, 2^50) (AR = 2): fp64 residues, each
// product an exact signed representative in (-q, q) from one fp64 product and its fma
// error term (fpmod.h), summed in doubles and brought back every six terms; the 24
// accumulators take a third of the registers of the integer forms, so five waves fit
// per SIMD instead of three.  All below 2^50 (AR = 1): a word w < 2^50 is split into
// w0 = w mod 2^25 and w1 = floor(w / 2^25), both below 2^25, and
//   x p = x0 p0 + (x0 p1 + x1 p0) 2^25 + x1 p1 2^50;
// the three partial sums are kept in 64-bit registers, each partial product added by one
// 32 x 32 + 64 multiply-add (every partial below 2^51, so GM_MAX_TERMS terms fit), and the
// group's sum is assembled to 128 bits and reduced once at the end.  Otherwise (AR = 0,
// wider primes) products are summed in 128 bits and reduced every four terms.
constexpr int GM_TB = 128;
constexpr int GM_MAX_TERMS = 8191;   // 64-bit partial sums: 8191 * 2^51 < 2^64

template <int NP, int AR>
__global__ void __launch_bounds__(GM_TB) k_group_mac_np(const MacTermNP* __restrict__ terms, const int* __restrict__ group_start,
                               uint64_t* const* __restrict__ outs, int l1, int accumulate, int log_n, int n_groups,
                               int xcd_order, const Mod* __restrict__ mods) {
  typedef uint64_t v2 __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(1))) const v2 gv2;
  typedef __attribute__((address_space(1))) v2 gv2w;
  const size_t N = (size_t)1 << log_n;
  const int i = blockIdx.z;
  int jb, g;
  if (xcd_order) {   // every group of one coefficient block back to back on one XCD
    const int b = blockIdx.x, idx = b >> 3;
    jb = (b & 7) + 8 * (idx / n_groups);
    g = idx % n_groups;
  } else {
    jb = blockIdx.x;
    g = blockIdx.y;
  }
  const size_t j = 2 * ((size_t)jb * GM_TB + threadIdx.x);
  const Mod m = mods[i];
  const size_t o0 = (size_t)i * N + j, o1 = ((size_t)l1 + i) * N + j;
  const int t_end = group_start[g + 1];
  int t = group_start[g];
  // per ciphertext, the four words of a thread: component 0 at j, j+1, component 1 at j, j+1
  uint64_t res[NP][4];
  if (AR == 2) {
    // fp64 residues (every prime in (2^49, 2^50)): each product a signed representative in
    // (-q, q), summed in a double; six terms at most between reductions keep every sum an
    // exact integer below 2^53
    const double qd = (double)m.q, qinv = m.qinv;
    double S[NP][4];
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) S[c][k] = 0.0;
    auto cv = [](uint64_t v) { return b2f(to_fbits(v)); };
    auto mac = [&](const v2& p, const v2 (&x)[NP], const v2 (&y)[NP]) {
      const double p0 = cv(p.x), p1 = cv(p.y);
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        S[c][0] += fmulmod_s(cv(x[c].x), p0, qd, qinv);
        S[c][1] += fmulmod_s(cv(x[c].y), p1, qd, qinv);
        S[c][2] += fmulmod_s(cv(y[c].x), p0, qd, qinv);
        S[c][3] += fmulmod_s(cv(y[c].y), p1, qd, qinv);
      }
    };
    auto fold = [&]() {
#pragma unroll
      for (int c = 0; c < NP; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) S[c][k] = sred(S[c][k], qd, qinv);
    };
    int cnt = 0;
    for (; t + 2 <= t_end; t += 2) {
      const MacTermNP ta = terms[t], tb = terms[t + 1];
      v2 pa = {1, 1}, pb = {1, 1};
      if (ta.pt) pa = __builtin_nontemporal_load((gv2*)(ta.pt + (size_t)i * N + j));
      if (tb.pt) pb = __builtin_nontemporal_load((gv2*)(tb.pt + (size_t)i * N + j));
      v2 xa[NP], ya[NP], xb[NP], yb[NP];
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        xa[c] = *(gv2*)(ta.ct[c] + o0);
        ya[c] = *(gv2*)(ta.ct[c] + o1);
        xb[c] = *(gv2*)(tb.ct[c] + o0);
        yb[c] = *(gv2*)(tb.ct[c] + o1);
      }
      mac(pa, xa, ya);
      mac(pb, xb, yb);
      if ((cnt += 2) == 6) {
        fold();
        cnt = 0;
      }
    }
    if (t < t_end) {
      const MacTermNP ta = terms[t];
      v2 pa = {1, 1};
      if (ta.pt) pa = __builtin_nontemporal_load((gv2*)(ta.pt + (size_t)i * N + j));
      v2 xa[NP], ya[NP];
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        xa[c] = *(gv2*)(ta.ct[c] + o0);
        ya[c] = *(gv2*)(ta.ct[c] + o1);
      }
      mac(pa, xa, ya);
    }
    fold();
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) res[c][k] = from_fbits(f2b(canon(S[c][k], qd)));
  } else if (AR == 1) {
    uint64_t A[NP][4], B[NP][4], C[NP][4];
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) A[c][k] = B[c][k] = C[c][k] = 0;
    auto part = [&](uint64_t& a, uint64_t& b, uint64_t& cc, uint64_t w, uint32_t p0, uint32_t p1) {
      const uint32_t w0 = (uint32_t)w & M25, w1 = (uint32_t)(w >> 25);
      a += (uint64_t)w0 * p0;
      b += (uint64_t)w0 * p1;
      b += (uint64_t)w1 * p0;
      cc += (uint64_t)w1 * p1;
    };
    auto mac = [&](const v2& p, const v2 (&x)[NP], const v2 (&y)[NP]) {
      const uint32_t px0 = (uint32_t)p.x & M25, px1 = (uint32_t)(p.x >> 25);
      const uint32_t py0 = (uint32_t)p.y & M25, py1 = (uint32_t)(p.y >> 25);
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        part(A[c][0], B[c][0], C[c][0], x[c].x, px0, px1);
        part(A[c][1], B[c][1], C[c][1], x[c].y, py0, py1);
        part(A[c][2], B[c][2], C[c][2], y[c].x, px0, px1);
        part(A[c][3], B[c][3], C[c][3], y[c].y, py0, py1);
      }
    };
    for (; t + 2 <= t_end; t += 2) {
      const MacTermNP ta = terms[t], tb = terms[t + 1];
      v2 pa = {1, 1}, pb = {1, 1};
      // each mask word is read once: streamed past the cache so that the baby-step words,
      // which every giant step of this coefficient block reads again, stay in L2
      if (ta.pt) pa = __builtin_nontemporal_load((gv2*)(ta.pt + (size_t)i * N + j));
      if (tb.pt) pb = __builtin_nontemporal_load((gv2*)(tb.pt + (size_t)i * N + j));
      v2 xa[NP], ya[NP], xb[NP], yb[NP];
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        xa[c] = *(gv2*)(ta.ct[c] + o0);
        ya[c] = *(gv2*)(ta.ct[c] + o1);
        xb[c] = *(gv2*)(tb.ct[c] + o0);
        yb[c] = *(gv2*)(tb.ct[c] + o1);
      }
      mac(pa, xa, ya);
      mac(pb, xb, yb);
    }
    if (t < t_end) {
      const MacTermNP ta = terms[t];
      v2 pa = {1, 1};
      if (ta.pt) pa = __builtin_nontemporal_load((gv2*)(ta.pt + (size_t)i * N + j));
      v2 xa[NP], ya[NP];
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        xa[c] = *(gv2*)(ta.ct[c] + o0);
        ya[c] = *(gv2*)(ta.ct[c] + o1);
      }
      mac(pa, xa, ya);
    }
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        res[c][k] = reduce128((u128)A[c][k] + ((u128)B[c][k] << 25) + ((u128)C[c][k] << 50), m);
  } else {
    u128 s[NP][4];
#pragma unroll
    for (int c = 0; c < NP; ++c) {
      res[c][0] = res[c][1] = res[c][2] = res[c][3] = 0;
      s[c][0] = s[c][1] = s[c][2] = s[c][3] = 0;
    }
    auto mac = [&](const v2& p, const v2 (&x)[NP], const v2 (&y)[NP]) {
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        s[c][0] += (u128)x[c].x * p.x;
        s[c][1] += (u128)x[c].y * p.y;
        s[c][2] += (u128)y[c].x * p.x;
        s[c][3] += (u128)y[c].y * p.y;
      }
    };
    auto fold = [&]() {
#pragma unroll
      for (int c = 0; c < NP; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          res[c][k] = add_mod(res[c][k], reduce128(s[c][k], m), m.q);
          s[c][k] = 0;
        }
    };
    // two terms' loads in flight together; products of four terms summed in 128 bits
    // (each below 2^124 for words below 2^62) before one reduction
    int cnt = 0;
    for (; t + 2 <= t_end; t += 2) {
      const MacTermNP ta = terms[t], tb = terms[t + 1];
      v2 pa = {1, 1}, pb = {1, 1};
      if (ta.pt) pa = *(gv2*)(ta.pt + (size_t)i * N + j);
      if (tb.pt) pb = *(gv2*)(tb.pt + (size_t)i * N + j);
      v2 xa[NP], ya[NP], xb[NP], yb[NP];
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        xa[c] = *(gv2*)(ta.ct[c] + o0);
        ya[c] = *(gv2*)(ta.ct[c] + o1);
        xb[c] = *(gv2*)(tb.ct[c] + o0);
        yb[c] = *(gv2*)(tb.ct[c] + o1);
      }
      mac(pa, xa, ya);
      mac(pb, xb, yb);
      if ((cnt += 2) == 4) {
        fold();
        cnt = 0;
      }
    }
    if (t < t_end) {
      const MacTermNP ta = terms[t];
      v2 pa = {1, 1};
      if (ta.pt) pa = *(gv2*)(ta.pt + (size_t)i * N + j);
      v2 xa[NP], ya[NP];
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        xa[c] = *(gv2*)(ta.ct[c] + o0);
        ya[c] = *(gv2*)(ta.ct[c] + o1);
      }
      mac(pa, xa, ya);
    }
    fold();
  }
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    uint64_t* out = outs[(size_t)g * NP + c];
    if (accumulate) {
      const v2 u = *(gv2*)(out + o0), v = *(gv2*)(out + o1);
      res[c][0] = add_mod(res[c][0], u.x, m.q);
      res[c][1] = add_mod(res[c][1], u.y, m.q);
      res[c][2] = add_mod(res[c][2], v.x, m.q);
      res[c][3] = add_mod(res[c][3], v.y, m.q);
    }
    const v2 r0 = {res[c][0], res[c][1]}, r1 = {res[c][2], res[c][3]};
    *(gv2w*)(out + o0) = r0;
    *(gv2w*)(out + o1) = r1;
  }
}

// ---- the same sums with the ciphertexts in LDS ----------------------------------------------
// Every giant step reads some of the same few baby-step ciphertexts, each a sixth of them at the
// 19717-node shape: there the sums above move 55 GB of ciphertext words from L2 for 9 GB of mask
// words, and L2 bounds them.  Here a workgroup takes 16 coefficients (128-byte runs) of one limb,
// reads those of every ciphertext into LDS once, as pairs of 25-bit halves, and walks all the
// groups: eight groups a wave, eight lanes a group, two coefficients a lane, so that a term is one
// 16-byte mask load and 2 NP 16-byte LDS reads.  With x = x0 + x1 2^25 and p alike, the sums of
// x0 p0, x1 p1 and (x0 + x1)(p0 + p1) are kept in 64 bits, three multiply-adds a product, no
// conversion, and reduced once a group (GL_MAX_TERMS bounds the third).  Groups go by falling
// length, so the eight of a wave end together, and a wave takes the next eight from a counter.
// Masks are requested eight terms ahead; the term list lies in LDS too, since loads come back in
// order and waiting for a list entry from memory would wait for every mask requested before it.
// Odd groups take the two components in the other order: at any time half of a wave reads each half
// of the LDS banks.
constexpr int GL_COEF = 16;
constexpr int GL_MAX_TERMS = 4095;     // 4095 * 2^52 < 2^64
constexpr int GL_MIN_TERMS = 3000;
constexpr int GL_T = 768;              // threads: three waves a SIMD, as the registers allow
// a term: the mask's place, in masks of l1 limbs from the base, and the ciphertext tuple
constexpr int GL_TUP_BITS = 9;
constexpr uint32_t GL_TUP = (1u << GL_TUP_BITS) - 1;
constexpr int GL_CAP = 6144;           // 96 KiB of ciphertext words
constexpr int GL_LIST = 12288;         // terms: 48 KiB
struct NpGroup {
  int32_t start, len, g;   // its terms, its number
};

template <int NP>
__global__ __launch_bounds__(GL_T) void k_group_mac_lds(
    const uint64_t* const* __restrict__ tuples, int n_tup, const uint32_t* __restrict__ terms, int n_terms,
    const NpGroup* __restrict__ groups, int n_groups, const uint64_t* __restrict__ pt_base,
    uint64_t* const* __restrict__ outs, int l1, int accumulate, int log_n, const Mod* __restrict__ mods,
    const Fold25* __restrict__ folds) {
  typedef uint64_t v2 __attribute__((ext_vector_type(2)));
  typedef uint32_t v4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(1))) const v2 gv2;
  typedef __attribute__((address_space(1))) v2 gv2w;
  constexpr int T = GL_T;
  constexpr int U = 4;                 // terms a step; masks are two steps ahead
  __shared__ v4 sx[GL_CAP];            // [tuple][NP][2 components][8 lanes]
  __shared__ uint32_t st[GL_LIST];
  __shared__ int ctr;
  const size_t N = (size_t)1 << log_n;
  const int i = blockIdx.y;
  const size_t j0 = (size_t)blockIdx.x * GL_COEF;
  auto halves = [](v2 w) {
    return v4{(uint32_t)w.x & M25, (uint32_t)(w.x >> 25), (uint32_t)w.y & M25, (uint32_t)(w.y >> 25)};
  };
  const int units = n_tup * NP * 2 * 8;
  for (int u = threadIdx.x; u < units; u += T) {
    const int lane = u & 7, comp = (u >> 3) & 1, tc = u >> 4;
    sx[u] = halves(*(gv2*)(tuples[tc] + ((size_t)comp * l1 + i) * N + j0 + 2 * lane));
  }
  for (int u = threadIdx.x; u < n_terms; u += T) st[u] = terms[u];
  if (threadIdx.x == 0) ctr = T / 64;
  __syncthreads();
  const int team = (threadIdx.x & 63) >> 3, l8 = threadIdx.x & 7;
  const Mod m = cld(mods + i);
  const uint64_t q = m.q;
  const bool fp = fp_prime(q);
  const double qd = (double)q;
  const Fold25 f = cld(folds + i);
  const IntQ iq = make_intq(q);
  const uint64_t* const mb = pt_base + (size_t)i * N + j0 + 2 * l8;
  const size_t mask_words = (size_t)l1 * N;
  const int odd = team & 1;
  const v4* const sl = sx + l8 + odd * 8;
  const int swap = odd ? -8 : 8;       // from a tuple's first component read to the other
  const int n_oct = (n_groups + 7) >> 3;
  auto mask = [&](uint32_t e) {
    return __builtin_nontemporal_load((gv2*)(mb + (size_t)(e >> GL_TUP_BITS) * mask_words));
  };
  int oct = threadIdx.x >> 6;
  while (oct < n_oct) {
    const int gi = oct * 8 + team;
    const NpGroup gd = gi < n_groups ? groups[gi] : NpGroup{0, 0, -1};
    // the longest of the eight (they go by falling length): the first
    const int n = __builtin_amdgcn_readfirstlane(groups[oct * 8].len);
    // a lane past its group's end repeats an entry (its last; the list's first where it has none)
    // and takes 0 for the mask
    const int first = gd.len > 0 ? gd.start : 0, last = gd.len > 0 ? gd.start + gd.len - 1 : 0;
    auto entry = [&](int t) { return st[first + t < last ? first + t : last]; };
    uint64_t A[NP][4], B[NP][4], C[NP][4];
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
      for (int k = 0; k < 4; ++k) A[c][k] = B[c][k] = C[c][k] = 0;
    uint32_t e[3][U];
    v2 p[3][U];
    // step s of the term loop uses e and p of slot s mod 3
    if (n > 0) {
#pragma unroll
      for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int u = 0; u < U; ++u) e[s][u] = entry(s * U + u);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int u = 0; u < U; ++u) p[s][u] = mask(e[s][u]);
    }
    auto step = [&](uint32_t (&ec)[U], v2 (&pc)[U], uint32_t (&en)[U], v2 (&pn)[U], int t) {
      // the masks two steps on, then this step's products, then the entries three steps on
#pragma unroll
      for (int u = 0; u < U; ++u) pn[u] = mask(en[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v2 pw = pc[u];
        if (t + u >= gd.len) pw = v2{0, 0};
        const v4 h = halves(pw);
        const uint32_t hs = h.x + h.y, ht = h.z + h.w;
        const v4* x = sl + (ec[u] & GL_TUP) * (NP * 16);
#pragma unroll
        for (int c = 0; c < NP; ++c)
#pragma unroll
          for (int comp = 0; comp < 2; ++comp) {
            const v4 w = x[c * 16 + (comp ? swap : 0)];
            const int k = comp * 2;
            A[c][k] += (uint64_t)w.x * h.x;
            C[c][k] += (uint64_t)w.y * h.y;
            B[c][k] += (uint64_t)(w.x + w.y) * hs;
            A[c][k + 1] += (uint64_t)w.z * h.z;
            C[c][k + 1] += (uint64_t)w.w * h.w;
            B[c][k + 1] += (uint64_t)(w.z + w.w) * ht;
          }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) ec[u] = entry(t + 3 * U + u);
    };
    if (n > 0)
      for (int t = 0;;) {
        step(e[0], p[0], e[2], p[2], t);
        if ((t += U) >= n) break;
        step(e[1], p[1], e[0], p[0], t);
        if ((t += U) >= n) break;
        step(e[2], p[2], e[1], p[1], t);
        if ((t += U) >= n) break;
      }
    if (gd.g >= 0) {
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        uint64_t* out = outs[(size_t)gd.g * NP + c] + (size_t)i * N + j0 + 2 * l8;
        uint64_t r[4];
        if (fp) {
#pragma unroll
          for (int w = 0; w < 4; ++w)
            r[w] = fold25_fp(A[c][w], B[c][w] - A[c][w] - C[c][w], C[c][w], qd, m.qinv, f);
        } else {
#pragma unroll
          for (int w = 0; w < 4; ++w) r[w] = fold25_int(A[c][w], B[c][w] - A[c][w] - C[c][w], C[c][w], q, iq, f);
        }
#pragma unroll
        for (int comp = 0; comp < 2; ++comp) {
          uint64_t* o = out + (size_t)(comp ^ odd) * mask_words;
          v2 v = {r[comp * 2], r[comp * 2 + 1]};
          if (accumulate) {
            const v2 old = *(gv2*)o;
            v.x = add_mod(v.x, old.x, q);
            v.y = add_mod(v.y, old.y, q);
          }
          *(gv2w*)o = v;
        }
      }
    }
    if ((threadIdx.x & 63) == 0) oct = atomicAdd(&ctr, 1);
    oct = __builtin_amdgcn_readfirstlane(oct);
  }
}

// One launch's groups as the LDS form reads them: as many of groups[g0..) as its tables hold, in the
// order of falling length.  Returns the first group left, or g0 where the form does not apply: one
// group's terms or distinct ciphertext tuples beyond the tables, terms without a mask, masks that are
// not whole masks apart.
struct LdsForm {
  std::vector<const uint64_t*> tuples;
  std::vector<uint32_t> terms;
  std::vector<NpGroup> groups;
  const uint64_t* base = nullptr;
};
static size_t lds_form(ckks_ctx* c, int level, int np, const std::vector<std::vector<MacTermNP>>& groups, size_t g0,
                       LdsForm& f) {
  const size_t mask_words = (size_t)(level + 1) * c->N;
  for (const auto& g : groups)
    for (const MacTermNP& t : g)
      if (t.pt && (!f.base || t.pt < f.base)) f.base = t.pt;
  std::map<std::vector<const uint64_t*>, uint32_t> seen;
  size_t g1 = g0;
  for (; g1 < groups.size(); ++g1) {
    const auto& g = groups[g1];
    if (g.size() > (size_t)GL_MAX_TERMS || f.terms.size() + g.size() > (size_t)GL_LIST) break;
    const size_t start = f.terms.size();
    bool fits = true;
    for (const MacTermNP& t : g) {
      const size_t w = (size_t)(t.pt - f.base);
      if (!t.pt || w % mask_words || w / mask_words >= (1u << (32 - GL_TUP_BITS))) return g0;
      const std::vector<const uint64_t*> key(t.ct, t.ct + np);
      auto it = seen.find(key);
      if (it == seen.end()) {
        fits = (seen.size() + 1) * np * 16 <= (size_t)GL_CAP && seen.size() < GL_TUP;
        if (!fits) break;
        it = seen.emplace(key, (uint32_t)seen.size()).first;
        f.tuples.insert(f.tuples.end(), key.begin(), key.end());
      }
      f.terms.push_back((uint32_t)(w / mask_words) << GL_TUP_BITS | it->second);
    }
    if (!fits) {
      f.terms.resize(start);
      break;
    }
    f.groups.push_back(NpGroup{(int32_t)start, (int32_t)g.size(), (int32_t)g1});
  }
  std::stable_sort(f.groups.begin(), f.groups.end(), [](const NpGroup& a, const NpGroup& b) { return a.len > b.len; });
  return g1;
}

void group_mac_np(ckks_ctx* c, int level, int np, const std::vector<std::vector<MacTermNP>>& groups,
                  const std::vector<uint64_t*>& outs, bool accumulate) {
  if (groups.empty()) return;
  if (np < 1 || np > MacTermNP::MAX) FICGCN_THROW(EINVAL_, "shared-mask sum: 1 to 4 ciphertexts per term");
  if (outs.size() != groups.size() * np) FICGCN_THROW(EINVAL_, "group/output count mismatch");
  if (c->N < 2 * GM_TB) FICGCN_THROW(EINVAL_, "ring too small for the shared-mask sum");
  std::vector<MacTermNP> flat;
  std::vector<int> start{0};
  for (const auto& g : groups) {
    for (const MacTermNP& t : g)
      for (int k = 0; k < np; ++k)
        if (!t.ct[k]) FICGCN_THROW(EINVAL_, "null term");
    flat.insert(flat.end(), g.begin(), g.end());
    start.push_back((int)flat.size());
  }
  for (uint64_t* o : outs)
    if (!o) FICGCN_THROW(EINVAL_, "null output");
  if (groups.size() > 65535) FICGCN_THROW(EINVAL_, "too many groups in one launch");
  const int n_jb = c->N / (2 * GM_TB), ng = (int)groups.size();
  const bool xcd = n_jb % 8 == 0 && (size_t)n_jb * ng < ((size_t)1 << 31);
  const dim3 grid = xcd ? dim3(n_jb * ng, 1, level + 1) : dim3(n_jb, ng, level + 1);
  const int acc = accumulate ? 1 : 0;
  // split-limb products need every prime of the level below 2^50 and at most GM_MAX_TERMS
  // terms per group
  bool l25 = true, f50 = true;
  for (int i = 0; i <= level; ++i) {
    l25 = l25 && c->mod[i] < (1ull << 50);
    f50 = f50 && c->mod[i] > (1ull << 49) && c->mod[i] < (1ull << 50);
  }
  for (size_t gi = 0; gi < groups.size(); ++gi) l25 = l25 && groups[gi].size() <= (size_t)GM_MAX_TERMS;
  const int ar = f50 ? 2 : l25 ? 1 : 0;
  // The LDS form where it is the faster one: two or three ciphertexts a term and GL_MIN_TERMS terms a
  // launch.  Measured at N = 2^16, level 2, against the form below (us): 5860 terms over three
  // ciphertexts 3040 for 4250, 3734 terms 2245 for 2826 (two ciphertexts 1937 for 2149, one 1714 for
  // 1609), 2062 terms 1787 for 1625 (two 1424 for 1233); with fewer terms its fixed cost, the
  // ciphertexts' way into LDS, shows, and those of few fit L2 anyway.  Four do not fit its tables.
  size_t g0 = 0;
  while (l25 && (np == 2 || np == 3) && flat.size() - start[g0] >= (size_t)GL_MIN_TERMS) {
    LdsForm f;
    const size_t g1 = lds_form(c, level, np, groups, g0, f);
    if (g1 == g0 || f.terms.size() < (size_t)GL_MIN_TERMS) break;
    const auto [tup, td, gd, od] = upload(c, S_GM_TERMS, f.tuples, f.terms, f.groups, outs);
    ProfScope ps(c, "bsgs_inner");   // the launch alone (its tables are uploaded above)
    const dim3 lgrid(c->N / GL_COEF, level + 1);
    const int n_tup = (int)(f.tuples.size() / np), nt = (int)f.terms.size(), nlg = (int)f.groups.size();
#define GL_LAUNCH(NPV)                                                                                            \
  hipLaunchKernelGGL(k_group_mac_lds<NPV>, lgrid, dim3(GL_T), 0, c->stream, tup, n_tup, td, nt, gd, nlg, \
                     f.base, od, level + 1, acc, c->log_n, c->t.mods, c->t.fold25)
    if (np == 2)
      GL_LAUNCH(2);
    else
      GL_LAUNCH(3);
#undef GL_LAUNCH
    HIPCHECK(hipGetLastError());
    ps.stop();
    g0 = g1;
  }
  if (g0) {   // the rest, if any, in the form below
    if (g0 == groups.size()) return;
    group_mac_np(c, level, np, std::vector<std::vector<MacTermNP>>(groups.begin() + g0, groups.end()),
                 std::vector<uint64_t*>(outs.begin() + g0 * np, outs.end()), accumulate);
    return;
  }
  const auto [td, sd, od] = upload(c, S_GM_TERMS, flat, start, outs);
  ProfScope ps(c, "bsgs_inner");   // the launch alone (its tables are uploaded above)
#define GM_LAUNCH(NPV, AV)                                                                                     \
  hipLaunchKernelGGL((k_group_mac_np<NPV, AV>), grid, dim3(GM_TB), 0, c->stream, td, sd, od, level + 1, acc, \
                     c->log_n, ng, xcd ? 1 : 0, c->t.mods)
#define GM_BY_AR(NPV)          \
  switch (ar) {                \
    case 0: GM_LAUNCH(NPV, 0); break; \
    case 1: GM_LAUNCH(NPV, 1); break; \
    default: GM_LAUNCH(NPV, 2);       \
  }
  switch (np) {
    case 1: GM_BY_AR(1); break;
    case 2: GM_BY_AR(2); break;
    case 3: GM_BY_AR(3); break;
    default: GM_BY_AR(4);
  }
#undef GM_BY_AR
#undef GM_LAUNCH
  HIPCHECK(hipGetLastError());
  ps.stop();
}

}  // namespace ficgcn
