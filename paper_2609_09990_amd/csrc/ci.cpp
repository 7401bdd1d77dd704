// Determinant-space view of MPS states and their (transition) 1-/2-RDMs (the
// device CI pipeline of Sec. III; conventions in ci.hpp).
//
// MPS -> CI.  The chain is cut at c = L/2.  Left of the cut every prefix of
// physical states (s_0 .. s_{c-1}) that reaches a sector q of bond c carries the
// row vector A_0[s_0] ... A_{c-1}[s_{c-1}]; right of it every suffix carries
// A_c[s_c] ... A_{L-1}[s_{L-1}].  Both families grow one site at a time as block
// GEMMs (all prefixes of one sector times one site block), and the amplitudes
// of sector q are the product P_q S_q^T of its prefix and suffix matrices, one
// GEMM per sector.  A determinant's string ranks split into a prefix part and a
// suffix part (the suffix's ranks counted after the prefix's electrons, fixed by
// q), and so does its sign, so a scatter kernel places every amplitude.
//
// RDMs.  With the excited copies T_x = E_rs |c> (x = r n + s) and T_{n^2} = |c>,
//   <bra| E_pq |ket> = <bra | T^ket_{pq}>,
//   <bra| E_pq E_rs |ket> = <E_qp bra | E_rs ket> = <T^bra_{qp} | T^ket_{rs}>,
// so one product G = T^bra (T^ket)^T of (n^2 + 1) rows over all determinants
// gives gamma, Gamma' = <E_pq E_rs> - d_qr gamma_ps and <bra|ket>.  The copies are
// formed inside the product (ci_gram.hip); its partial sums over ranges of
// determinants are added in a fixed order (deterministic).
#include <algorithm>
#include <cmath>

#include "ci.hpp"
#include "solver.hpp"

namespace dmrg {
namespace {

long binom(int n, int k) {
  if (k < 0 || k > n) return 0;
  long r = 1;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}

int popc(uint32_t x) { return __builtin_popcount(x); }

// Colexicographic rank contribution of the occupied orbitals of `bits`, the
// first of them being electron number t0 of its spin.
long colex_part(uint32_t bits, int t0) {
  long r = 0;
  int t = t0;
  for (int o = 0; o < 32; ++o)
    if (bits >> o & 1u) r += binom(o, ++t);
  return r;
}

std::vector<uint32_t> colex_strings(int n, int k) {
  std::vector<uint32_t> out(binom(n, k));
  for (uint32_t m = 0; m < (1u << n); ++m)
    if (popc(m) == k) out[colex_part(m, 0)] = m;
  return out;
}

// The excitation tables of one spin's strings (ci.hpp; `unit`: N_b for alpha, 1 for
// beta strings): a_s removes s from I with (-1)^(electrons below s), a+_r inserts r
// into what is left with (-1)^(electrons below r).
std::vector<int> excitation_table(int n, const std::vector<uint32_t>& strs, long unit, bool identity) {
  const long N = (long)strs.size();
  std::vector<int> rank((size_t)1 << n, -1);
  for (long J = 0; J < N; ++J) rank[strs[J]] = (int)J;
  std::vector<int> t(((long)n * n + 2) * N, 0);
  for (long J = 0; J < N; ++J) {
    const uint32_t j = strs[J];
    for (int r = 0; r < n; ++r) {
      if (!(j >> r & 1u)) continue;
      for (int s = 0; s < n; ++s) {
        if (s != r && (j >> s & 1u)) continue;
        const uint32_t i = (j & ~(1u << r)) | (1u << s);
        const uint32_t i1 = i & ~(1u << s);
        const int par = popc(i & ((1u << s) - 1)) + popc(i1 & ((1u << r) - 1));
        const int I = (int)(rank[i] * unit) + 1;
        t[((long)r * n + s) * N + J] = (par & 1) ? -I : I;
      }
    }
    if (identity) t[(long)n * n * N + J] = (int)(J * unit) + 1;
  }
  return t;
}

void tiles64(std::vector<GemmUnit>& units, double* C, int ldc, int M, int N, int ib, int ie) {
  for (int m0 = 0; m0 < M; m0 += 64)
    for (int n0 = 0; n0 < N; n0 += 64) units.push_back({C, ldc, M, N, m0, n0, ib, ie, 0});
}

// one generic-kernel GEMM launch over 64 x 64 tiles (items and units uploaded here)
void gemm_tiles(int mode, const std::vector<GemmItem>& items, const std::vector<GemmUnit>& units, hipStream_t st);

template <class T>
void upload(DevMem& d, const std::vector<T>& v, hipStream_t st) {
  d.reserve(std::max<size_t>(v.size(), 1) * sizeof(T));
  if (!v.empty()) hip_check(hipMemcpyAsync(d.p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, st), "ci upload");
}

// rank of every n-bit mask among the strings with k bits, -1 for the others
std::vector<int> rank_table(int n, int k) {
  std::vector<int> r((size_t)1 << n, -1);
  for (uint32_t m = 0; m < (1u << n); ++m)
    if (popc(m) == k) r[m] = (int)colex_part(m, 0);
  return r;
}

// Eigenvalues (ascending) and, if V, eigenvectors (columns of the row-major
// n x n V) of a symmetric matrix by cyclic Jacobi rotations (small n only).
void jacobi_eigh(std::vector<double> A, int n, std::vector<double>& w, std::vector<double>* V) {
  std::vector<double> Q((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) Q[(size_t)i * n + i] = 1.0;
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0, tot = 0;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) {
        tot += A[(size_t)i * n + j] * A[(size_t)i * n + j];
        if (i != j) off += A[(size_t)i * n + j] * A[(size_t)i * n + j];
      }
    if (off <= 1e-30 * std::max(tot, 1e-300)) break;
    for (int p = 0; p < n; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = A[(size_t)p * n + q];
        if (apq == 0.0) continue;
        const double th = (A[(size_t)q * n + q] - A[(size_t)p * n + p]) / (2 * apq);
        const double t = (th >= 0 ? 1.0 : -1.0) / (std::fabs(th) + std::sqrt(th * th + 1));
        const double cs = 1 / std::sqrt(t * t + 1), sn = t * cs;
        for (int k = 0; k < n; ++k) {  // columns p, q
          const double akp = A[(size_t)k * n + p], akq = A[(size_t)k * n + q];
          A[(size_t)k * n + p] = cs * akp - sn * akq;
          A[(size_t)k * n + q] = sn * akp + cs * akq;
        }
        for (int k = 0; k < n; ++k) {  // rows p, q
          const double apk = A[(size_t)p * n + k], aqk = A[(size_t)q * n + k];
          A[(size_t)p * n + k] = cs * apk - sn * aqk;
          A[(size_t)q * n + k] = sn * apk + cs * aqk;
        }
        for (int k = 0; k < n; ++k) {
          const double qkp = Q[(size_t)k * n + p], qkq = Q[(size_t)k * n + q];
          Q[(size_t)k * n + p] = cs * qkp - sn * qkq;
          Q[(size_t)k * n + q] = sn * qkp + cs * qkq;
        }
      }
  }
  std::vector<int> idx(n);
  for (int i = 0; i < n; ++i) idx[i] = i;
  std::stable_sort(idx.begin(), idx.end(),
                   [&](int a, int b) { return A[(size_t)a * n + a] < A[(size_t)b * n + b]; });
  w.resize(n);
  for (int i = 0; i < n; ++i) w[i] = A[(size_t)idx[i] * n + idx[i]];
  if (V) {
    V->assign((size_t)n * n, 0.0);
    for (int i = 0; i < n; ++i)
      for (int k = 0; k < n; ++k) (*V)[(size_t)k * n + i] = Q[(size_t)k * n + idx[i]];
  }
}

double entropy_of(const std::vector<double>& rho, int n) {
  std::vector<double> w;
  jacobi_eigh(rho, n, w, nullptr);
  double s = 0;
  for (double x : w)
    if (x > 1e-300) s -= x * std::log(x);
  return s;
}

void gemm_tiles(int mode, const std::vector<GemmItem>& items, const std::vector<GemmUnit>& units, hipStream_t st) {
  if (units.empty()) return;
  DevMem di, du;
  upload(di, items, st);
  upload(du, units, st);
  launch_gemm(PREC_F64, mode, du.as<GemmUnit>(), (int)units.size(), di.as<GemmItem>(), st);
  hip_check(hipStreamSynchronize(st), "ci gemm");
}

// A checked-out set of tables and scratch: from the problem's pool, or (in a
// workspace, whose memory must not outlive the call, or without a pool) its own.
class Work {
 public:
  Work(CiPool* pool, int n, int na, int nb, hipStream_t st) : pool_(current_arena() ? nullptr : pool), st_(st) {
    w_ = pool_ ? pool_->take() : std::make_unique<CiWork>();
    if (!w_->tables) {
      const std::vector<uint32_t> sa = colex_strings(n, na), sb = colex_strings(n, nb);
      const std::vector<int> a = excitation_table(n, sa, (long)sb.size(), true), b = excitation_table(n, sb, 1, false);
      upload(w_->ta, a, st);
      upload(w_->tb, b, st);
      hip_check(hipStreamSynchronize(st), "excitation tables");
      w_->tables = true;
    }
  }
  ~Work() {
    (void)hipStreamSynchronize(st_);  // nothing of this call still uses the set
    if (pool_) pool_->give(std::move(w_));
  }
  Work(const Work&) = delete;
  Work& operator=(const Work&) = delete;
  CiWork* operator->() { return w_.get(); }

 private:
  CiPool* pool_;
  hipStream_t st_;
  std::unique_ptr<CiWork> w_;
};

// G (m x n) of the A and B rows of `src_a`, `src_b` into w->G (one list, src_a and
// rows `a`, when symmetric).
void gram(Work& w, int n, bool sym, const double* src_a, std::vector<GramRow> a, const double* src_b, std::vector<GramRow> b,
          long NA, long NB, hipStream_t st) {
  GramArgs P{};
  P.m = (int)a.size();
  P.n = sym ? P.m : (int)b.size();
  P.zero = n * n + 1;
  auto pad = [&](std::vector<GramRow>& v) {
    while (v.size() % 16) v.push_back({0, P.zero, 0});
  };
  pad(a);
  pad(b);
  const int ba = (int)a.size() / 16, bb = (int)b.size() / 16;
  std::vector<GramGroup> groups;
  std::vector<int2> pairs;
  int max_pairs = 0, max_rows = 0;
  if (sym) {
    DMRG_REQUIRE(ba <= 17, ST_EINVAL, "too many rows of a symmetric product");
    for (int i = 0; i < ba; ++i)
      for (int j = 0; j <= i; ++j) pairs.push_back({i, j});
    groups.push_back({0, 0, 0, (int)pairs.size()});
    max_pairs = (int)pairs.size();
    max_rows = 16 * ba;
  } else {
    DMRG_REQUIRE(ba <= 17, ST_EINVAL, "too many rows of a product");
    for (int b0 = 0; b0 < bb; b0 += kGramRows / 16) {
      const int nb = std::min(kGramRows / 16, bb - b0), p0 = (int)pairs.size();
      for (int i = 0; i < ba; ++i)
        for (int j = 0; j < nb; ++j) pairs.push_back({i, j});
      groups.push_back({16 * b0, 16 * nb, p0, (int)pairs.size() - p0});
      max_pairs = std::max(max_pairs, ba * nb);
      max_rows = std::max(max_rows, 16 * (ba + nb));
    }
  }
  P.src_a = src_a;
  P.src_b = src_b;
  P.ta = w->ta.as<int>();
  P.tb = w->tb.as<int>();
  P.na = (int)NA;
  P.nb = (int)NB;
  P.ndet = NA * NB;
  P.rows_a = 16 * ba;
  P.sym = sym;
  // Ranges of determinants: two workgroups per CU for one group of blocks, at most
  // four rounds of one per CU for many, at least two slices of 32 each.
  const long slices = (P.ndet + 31) / 32, ng = (long)groups.size();
  const int nsplit = (int)std::max<long>(1, std::min<long>(ng == 1 ? 512 : std::max<long>(1, 1024 / ng), slices / 2));
  // tables back to back in one buffer
  const size_t sa = a.size() * sizeof(GramRow), sb = b.size() * sizeof(GramRow), sg = groups.size() * sizeof(GramGroup),
               sp = pairs.size() * sizeof(int2);
  std::vector<char> h(sa + sb + sg + sp);
  std::copy((const char*)a.data(), (const char*)a.data() + sa, h.data());
  std::copy((const char*)b.data(), (const char*)b.data() + sb, h.data() + sa);
  std::copy((const char*)groups.data(), (const char*)groups.data() + sg, h.data() + sa + sb);
  std::copy((const char*)pairs.data(), (const char*)pairs.data() + sp, h.data() + sa + sb + sg);
  w->part.reserve((size_t)nsplit * pairs.size() * 256 * 8);
  w->G.reserve((size_t)P.m * P.n * 8);
  w->lists.reserve(h.size());
  hip_check(hipMemcpyAsync(w->lists.p, h.data(), h.size(), hipMemcpyHostToDevice, st), "gram tables");
  char* d = w->lists.as<char>();
  P.list_a = (const GramRow*)d;
  P.list_b = (const GramRow*)(d + sa);
  P.groups = (const GramGroup*)(d + sa + sb);
  P.pairs = (const int2*)(d + sa + sb + sg);
  P.partial = w->part.as<double>();
  P.G = w->G.as<double>();
  launch_gram(P, (int)groups.size(), (int)pairs.size(), max_pairs, max_rows, nsplit, st);
  hip_check(hipStreamSynchronize(st), "gram");  // h is read
}

}  // namespace

long ci_dimension(int n, int na, int nb) { return binom(n, na) * binom(n, nb); }

std::unique_ptr<CiWork> CiPool::take() {
  int dev = 0;
  hip_check(hipGetDevice(&dev), "device");
  {
    std::lock_guard<std::mutex> l(m_);
    for (size_t i = 0; i < idle_.size(); ++i)
      if (idle_[i]->device == dev) {
        std::unique_ptr<CiWork> w = std::move(idle_[i]);
        idle_.erase(idle_.begin() + i);
        return w;
      }
  }
  auto w = std::make_unique<CiWork>();
  w->device = dev;
  return w;
}

void CiPool::give(std::unique_ptr<CiWork> w) {
  // the largest buffers go first when the set is over the bound
  for (;;) {
    size_t sum = 0;
    DevMem* big = nullptr;
    for (DevMem* d : w->scratch()) {
      sum += d->bytes;
      if (!big || d->bytes > big->bytes) big = d;
    }
    if (sum <= kKeep) break;
    big->release();
  }
  std::lock_guard<std::mutex> l(m_);
  if (idle_.size() < 2) idle_.push_back(std::move(w));
}

void CiPool::drop() {
  std::lock_guard<std::mutex> l(m_);
  idle_.clear();
}

// V c with V = 1/2 sum_pqrs (pq|rs) E_pq E_rs and (pq|rs) = sum_Q B^Q_pq B^Q_rs,
// streamed through the factors: T_rs = E_rs c, W_Q = sum_rs B^Q_rs T_rs,
// U_pq = sum_Q B^Q_pq W_Q (one kernel, T and W on chip), V c = 1/2 sum_pq E_pq
// U_pq (a gather); (pq|rs) is never formed.
void ci_apply_v(CiPool* pool, int n, int na, int nb, int nq, const double* Bh, hipStream_t st, const double* c,
                double* out) {
  DMRG_REQUIRE(n >= 1 && n <= 16 && nq >= 0, ST_EINVAL, "the two-electron operator on CI vectors needs 1..16 orbitals");
  const long NA = binom(n, na), NB = binom(n, nb), N = NA * NB;
  const int n2 = n * n;
  if (nq == 0) {
    launch_fill(out, N, 0.0, st);
    hip_check(hipStreamSynchronize(st), "apply V");
    return;
  }
  Work w(pool, n, na, nb, st);
  w->T1.reserve((size_t)n2 * N * 8);
  w->F.reserve((size_t)nq * n2 * 8);
  hip_check(hipMemcpyAsync(w->F.p, Bh, (size_t)nq * n2 * 8, hipMemcpyHostToDevice, st), "B");
  double* U = w->T1.as<double>();
  launch_ci_uv(c, (int)NA, (int)NB, n2, nq, w->ta.as<int>(), w->tb.as<int>(), w->F.as<double>(), U, N, st);
  launch_ci_apply_sum(U, N, NA, NB, n2, w->ta.as<int>(), w->tb.as<int>(), 0.5, out, N, st);
  hip_check(hipStreamSynchronize(st), "apply V");
}

// Gamma3[pqrstu] = scale <bra|E_pq E_rs E_tu|ket> = scale <E_qp bra | E_rs E_tu ket>:
// the copies E_qp bra and E_tu ket are kept whole, E_rs of the latter is formed
// inside one product of n^2 bra rows with the n^2 (n^2 + 1) / 2 ket rows rs >= tu
// and the n^2 rows E_x ket, which give the others by the commutator.
void ci_rdm3(CiPool* pool, int n, int na, int nb, hipStream_t st, const double* bra, const double* ket, double scale,
             double* out) {
  DMRG_REQUIRE(n >= 1 && n <= 12, ST_EINVAL, "the three-body density from CI vectors needs 1..12 orbitals");
  const long NA = binom(n, na), NB = binom(n, nb), N = NA * NB;
  const int n2 = n * n;
  Work w(pool, n, na, nb, st);
  const bool same = bra == ket;
  w->T2.reserve((size_t)n2 * N * 8);
  if (!same) w->T1.reserve((size_t)n2 * N * 8);
  launch_ci_excite(ket, NA, NB, n2, w->ta.as<int>(), w->tb.as<int>(), w->T2.as<double>(), st);
  if (!same) launch_ci_excite(bra, NA, NB, n2, w->ta.as<int>(), w->tb.as<int>(), w->T1.as<double>(), st);
  std::vector<GramRow> a, b;
  for (int x = 0; x < n2; ++x) a.push_back({(long)x * N, n2, 0});
  // source by source: the rows of a group gather from one to three vectors, which
  // stay in L1 (excitation by excitation it would be 128)
  for (int y = 0; y < n2; ++y)
    for (int x = y; x < n2; ++x) b.push_back({(long)y * N, x, 0});
  for (int x = 0; x < n2; ++x) b.push_back({(long)x * N, n2, 0});
  gram(w, n, false, same ? w->T2.as<double>() : w->T1.as<double>(), std::move(a), w->T2.as<double>(), std::move(b), NA, NB,
       st);
  const long n6 = (long)n2 * n2 * n2;
  w->out.reserve((size_t)n6 * 8);
  launch_rdm3_assemble(w->G.as<double>(), n, scale, w->out.as<double>(), st);
  hip_check(hipMemcpyAsync(out, w->out.p, (size_t)n6 * 8, hipMemcpyDeviceToHost, st), "rdm3 out");
  hip_check(hipStreamSynchronize(st), "rdm3");
}

void orbital_rdm2(int n, int na, int nb, hipStream_t st, const double* c, std::vector<double>& rho) {
  DMRG_REQUIRE(n >= 2 && n <= 16, ST_EINVAL, "orbital density matrices from CI vectors need 2..16 orbitals");
  const std::vector<uint32_t> sa = colex_strings(n, na), sb = colex_strings(n, nb);
  const long NB = (long)sb.size(), N = (long)sa.size() * NB;
  std::vector<int> pairs;
  for (int i = 0; i < n; ++i)
    for (int j = i + 1; j < n; ++j) {
      pairs.push_back(i);
      pairs.push_back(j);
    }
  const int np = (int)pairs.size() / 2;
  const int nblk = (int)std::max<long>(1, std::min<long>((N + 255) / 256, (2048 + np - 1) / np));
  DevMem dsa, dsb, dra, drb, dpairs, part, out;
  upload(dsa, sa, st);
  upload(dsb, sb, st);
  upload(dra, rank_table(n, na), st);
  upload(drb, rank_table(n, nb), st);
  upload(dpairs, pairs, st);
  part.reserve((size_t)np * nblk * 36 * 8);
  out.reserve((size_t)np * 36 * 8);
  launch_orb_pairs(c, dsa.as<uint32_t>(), dsb.as<uint32_t>(), dra.as<int>(), drb.as<int>(), NB, N, dpairs.as<int>(), np,
                   nblk, part.as<double>(), st);
  launch_orb_sum(part.as<double>(), np, nblk, out.as<double>(), st);
  std::vector<double> e((size_t)np * 36);
  hip_check(hipMemcpyAsync(e.data(), out.p, e.size() * 8, hipMemcpyDeviceToHost, st), "orbital rdm");
  hip_check(hipStreamSynchronize(st), "orbital rdm");
  // expand the 36 entries of each pair: block (k_alpha, k_beta), states
  // (alpha configuration, beta configuration) in the kernel's order
  rho.assign((size_t)np * 256, 0.0);
  static const int kOff[9] = {0, 1, 5, 6, 10, 26, 30, 31, 35};
  for (int p = 0; p < np; ++p) {
    double* R = rho.data() + (size_t)p * 256;
    double tr = 0;
    for (int ka = 0; ka < 3; ++ka)
      for (int kb = 0; kb < 3; ++kb) {
        const int nA = ka == 1 ? 2 : 1, nB = kb == 1 ? 2 : 1, q = nA * nB;
        int L[4];
        for (int pa = 0; pa < nA; ++pa)
          for (int pb = 0; pb < nB; ++pb) {
            const int ai = ka == 2 || (ka == 1 && pa == 0), aj = ka == 2 || (ka == 1 && pa == 1);
            const int bi = kb == 2 || (kb == 1 && pb == 0), bj = kb == 2 || (kb == 1 && pb == 1);
            L[pa * nB + pb] = (ai + 2 * bi) + 4 * (aj + 2 * bj);
          }
        for (int x = 0; x < q; ++x)
          for (int y = 0; y < q; ++y) R[L[x] * 16 + L[y]] = e[(size_t)p * 36 + kOff[3 * ka + kb] + x * q + y];
        for (int x = 0; x < q; ++x) tr += R[L[x] * 16 + L[x]];
      }
    DMRG_REQUIRE(tr > 0, ST_EINVAL, "zero CI vector");
    for (int x = 0; x < 256; ++x) R[x] /= tr;
  }
}

void mutual_information(int n, int na, int nb, hipStream_t st, const double* c, double* s1, double* I) {
  std::vector<double> rho;
  orbital_rdm2(n, na, nb, st, c, rho);
  mutual_information_of(n, rho, s1, I);
}

void mutual_information_of(int n, const std::vector<double>& rho, double* s1, double* I) {
  std::vector<double> s2((size_t)n * n, 0.0);
  std::vector<double> one(n, -1.0);
  int p = 0;
  for (int i = 0; i < n; ++i)
    for (int j = i + 1; j < n; ++j, ++p) {
      const std::vector<double> R(rho.begin() + (size_t)p * 256, rho.begin() + (size_t)(p + 1) * 256);
      s2[(size_t)i * n + j] = entropy_of(R, 16);
      if (one[i] < 0 || one[j] < 0) {  // one-orbital matrices: diagonal partial traces
        double di[4] = {0, 0, 0, 0}, dj[4] = {0, 0, 0, 0};
        for (int L = 0; L < 16; ++L) {
          di[L % 4] += R[L * 16 + L];
          dj[L / 4] += R[L * 16 + L];
        }
        auto h = [](const double* d) {
          double s = 0;
          for (int t = 0; t < 4; ++t)
            if (d[t] > 1e-300) s -= d[t] * std::log(d[t]);
          return s;
        };
        if (one[i] < 0) one[i] = h(di);
        if (one[j] < 0) one[j] = h(dj);
      }
    }
  for (int i = 0; i < n; ++i) {
    s1[i] = one[i];
    I[(size_t)i * n + i] = 0;
    for (int j = i + 1; j < n; ++j)
      I[(size_t)i * n + j] = I[(size_t)j * n + i] = 0.5 * (one[i] + one[j] - s2[(size_t)i * n + j]);
  }
}

void fiedler_order(int n, const double* I, int* order, double* fiedler) {
  DMRG_REQUIRE(n >= 2 && n <= 64, ST_EINVAL, "ordering needs 2..64 orbitals");
  std::vector<double> Lap((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i) {
    double d = 0;
    for (int j = 0; j < n; ++j)
      if (j != i) {
        Lap[(size_t)i * n + j] = -I[(size_t)i * n + j];
        d += I[(size_t)i * n + j];
      }
    Lap[(size_t)i * n + i] = d;
  }
  std::vector<double> w, V;
  jacobi_eigh(Lap, n, w, &V);
  std::vector<double> v(n);
  int big = 0;
  for (int i = 0; i < n; ++i) {
    v[i] = V[(size_t)i * n + 1];
    if (std::fabs(v[i]) > std::fabs(v[big])) big = i;
  }
  if (v[big] < 0)
    for (double& x : v) x = -x;
  std::vector<int> idx(n);
  for (int i = 0; i < n; ++i) idx[i] = i;
  std::stable_sort(idx.begin(), idx.end(), [&](int a, int b) { return v[a] < v[b]; });
  for (int i = 0; i < n; ++i) {
    order[i] = idx[i];
    if (fiedler) fiedler[i] = v[i];
  }
}

void Solver::mps_to_ci(int state, double* c) {
  DMRG_REQUIRE(state >= 0 && state <= (int)defl_.size(), ST_EINVAL, "state must be 0 (this MPS) or a held state");
  const std::vector<Bond>& B = state == 0 ? bonds_ : defl_[state - 1].bonds;
  const std::vector<SiteTensor>& S = state == 0 ? mps_ : defl_[state - 1].sites;
  const int L = prob_->n;
  DMRG_REQUIRE((int)S.size() == L && (int)B.size() == L + 1, ST_ESTATE, "no MPS");
  DMRG_REQUIRE(L <= 24, ST_EINVAL, "the CI vector is built for at most 24 orbitals");
  const long Nb = binom(L, prob_->n_beta);
  DMRG_REQUIRE(ci_dimension(L, prob_->n_alpha, prob_->n_beta) < (1L << 31), ST_EINVAL, "CI space too large");
  DMRG_REQUIRE(B[0].sec.size() == 1 && B[0].sec[0].dim == 1 && B[L].sec.size() == 1 && B[L].sec[0].dim == 1,
               ST_ESTATE, "boundary bonds must hold one state");
  const int cut = L / 2;
  struct Str {
    uint32_t a, b;
  };
  struct Part {
    int src, dst;
    long r0;
    const double* blk;
    int ldb;
  };
  const double one = 1.0;
  std::vector<GemmItem> items;
  std::vector<GemmUnit> units;
  // prefixes: sites 0 .. cut-1, one matrix (prefixes x sector dim) per sector
  std::vector<std::vector<Str>> pre(1, std::vector<Str>{{0u, 0u}});
  std::vector<long> poff(1, 0);
  DevMem P, Pn;
  P.reserve(8);
  hip_check(hipMemcpyAsync(P.p, &one, 8, hipMemcpyHostToDevice, st), "ci");
  for (int k = 0; k < cut; ++k) {
    const Bond& bl = B[k];
    const Bond& br = B[k + 1];
    const SiteTensor& A = S[k];
    std::vector<std::vector<Str>> npre(br.sec.size());
    std::vector<Part> parts;
    for (size_t i = 0; i < bl.sec.size(); ++i) {
      if (pre[i].empty() || A.lay.slab_of_left[i] < 0) continue;
      const Slab& sb = A.lay.slabs[A.lay.slab_of_left[i]];
      for (int s = 0; s < 4; ++s) {
        const int j = br.find(bl.sec[i].q + site_qn(s));
        const int bi = j < 0 ? -1 : sb.block_of(s, j);
        if (bi < 0) continue;
        parts.push_back({(int)i, j, (long)npre[j].size(), A.buf.as<double>() + sb.off + sb.blocks[bi].col0, sb.width});
        for (const Str& p : pre[i]) npre[j].push_back({p.a | (uint32_t)(s & 1) << k, p.b | (uint32_t)(s >> 1) << k});
      }
    }
    std::vector<long> noff(br.sec.size(), 0);
    long tot = 0;
    for (size_t j = 0; j < br.sec.size(); ++j) {
      noff[j] = tot;
      tot += (long)npre[j].size() * br.sec[j].dim;
    }
    Pn.reserve(std::max<long>(tot, 1) * 8);
    items.clear();
    units.clear();
    for (const Part& pt : parts) {
      const int di = bl.sec[pt.src].dim, dj = br.sec[pt.dst].dim;
      const int ib = (int)items.size();
      items.push_back({P.as<double>() + poff[pt.src], pt.blk, di, pt.ldb, di, 0, 1.0});
      tiles64(units, Pn.as<double>() + noff[pt.dst] + pt.r0 * dj, dj, (int)pre[pt.src].size(), dj, ib, ib + 1);
    }
    gemm_once(GEMM_NN, items, units);
    std::swap(P, Pn);
    pre.swap(npre);
    poff.swap(noff);
  }
  // suffixes: sites cut .. L-1, one matrix (suffixes x sector dim) per sector
  std::vector<std::vector<Str>> suf(1, std::vector<Str>{{0u, 0u}});
  std::vector<long> soff(1, 0);
  DevMem Sm, Sn;
  Sm.reserve(8);
  hip_check(hipMemcpyAsync(Sm.p, &one, 8, hipMemcpyHostToDevice, st), "ci");
  for (int k = L - 1; k >= cut; --k) {
    const Bond& bl = B[k];
    const Bond& br = B[k + 1];
    const SiteTensor& A = S[k];
    std::vector<std::vector<Str>> nsuf(bl.sec.size());
    std::vector<Part> parts;
    for (size_t j = 0; j < br.sec.size(); ++j) {
      if (suf[j].empty()) continue;
      for (int s = 0; s < 4; ++s) {
        const int i = bl.find(br.sec[j].q - site_qn(s));
        if (i < 0 || A.lay.slab_of_left[i] < 0) continue;
        const Slab& sb = A.lay.slabs[A.lay.slab_of_left[i]];
        const int bi = sb.block_of(s, (int)j);
        if (bi < 0) continue;
        parts.push_back({(int)j, i, (long)nsuf[i].size(), A.buf.as<double>() + sb.off + sb.blocks[bi].col0, sb.width});
        for (const Str& x : suf[j]) nsuf[i].push_back({x.a | (uint32_t)(s & 1) << k, x.b | (uint32_t)(s >> 1) << k});
      }
    }
    std::vector<long> noff(bl.sec.size(), 0);
    long tot = 0;
    for (size_t i = 0; i < bl.sec.size(); ++i) {
      noff[i] = tot;
      tot += (long)nsuf[i].size() * bl.sec[i].dim;
    }
    Sn.reserve(std::max<long>(tot, 1) * 8);
    items.clear();
    units.clear();
    for (const Part& pt : parts) {
      const int dj = br.sec[pt.src].dim, di = bl.sec[pt.dst].dim;
      const int ib = (int)items.size();
      items.push_back({Sm.as<double>() + soff[pt.src], pt.blk, dj, pt.ldb, dj, 0, 1.0});
      tiles64(units, Sn.as<double>() + noff[pt.dst] + pt.r0 * di, di, (int)suf[pt.src].size(), di, ib, ib + 1);
    }
    gemm_once(GEMM_NT, items, units);
    std::swap(Sm, Sn);
    suf.swap(nsuf);
    soff.swap(noff);
  }
  // amplitudes per sector of the cut, rank and sign tables, scatter
  const Bond& bc = B[cut];
  std::vector<CiSector> secs;
  std::vector<int> pa, pb, sa, sb;
  std::vector<double> ps, ss;
  long amp = 0;
  items.clear();
  units.clear();
  std::vector<std::pair<size_t, long>> amp_at;
  for (size_t i = 0; i < bc.sec.size(); ++i) {
    const long np = (long)pre[i].size(), ns = (long)suf[i].size();
    if (np == 0 || ns == 0) continue;
    const QN q = bc.sec[i].q;
    const int a0 = (q.n + q.sz) / 2, b0 = (q.n - q.sz) / 2;
    secs.push_back({amp, (long)pa.size(), (long)sa.size(), (int)np, (int)ns});
    for (const Str& p : pre[i]) {
      int par = 0;
      for (int o = 0; o < cut; ++o)
        if (p.a >> o & 1u) par += popc(p.b & ((1u << o) - 1));
      pa.push_back((int)colex_part(p.a, 0));
      pb.push_back((int)colex_part(p.b, 0));
      ps.push_back(par & 1 ? -1.0 : 1.0);
    }
    for (const Str& x : suf[i]) {
      int par = popc(x.a) * b0;
      for (int o = cut; o < L; ++o)
        if (x.a >> o & 1u) par += popc(x.b & ((1u << o) - 1));
      sa.push_back((int)colex_part(x.a, a0));
      sb.push_back((int)colex_part(x.b, b0));
      ss.push_back(par & 1 ? -1.0 : 1.0);
    }
    amp_at.push_back({i, amp});
    amp += np * ns;
  }
  DevMem Amp;
  Amp.reserve(std::max<long>(amp, 1) * 8);
  for (const auto& [i, off] : amp_at) {
    const int d = bc.sec[i].dim, np = (int)pre[i].size(), ns = (int)suf[i].size();
    const int ib = (int)items.size();
    items.push_back({P.as<double>() + poff[i], Sm.as<double>() + soff[i], d, d, d, 0, 1.0});
    tiles64(units, Amp.as<double>() + off, ns, np, ns, ib, ib + 1);
  }
  gemm_once(GEMM_NT, items, units);
  DevMem dsec, dpa, dpb, dps, dsa, dsb, dss;
  upload(dsec, secs, st);
  upload(dpa, pa, st);
  upload(dpb, pb, st);
  upload(dps, ps, st);
  upload(dsa, sa, st);
  upload(dsb, sb, st);
  upload(dss, ss, st);
  launch_fill(c, ci_dimension(L, prob_->n_alpha, prob_->n_beta), 0.0, st);
  launch_ci_scatter(Amp.as<double>(), dsec.as<CiSector>(), (int)secs.size(), dpa.as<int>(), dpb.as<int>(),
                    dps.as<double>(), dsa.as<int>(), dsb.as<int>(), dss.as<double>(), c, Nb, st);
  hip_check(hipStreamSynchronize(st), "mps_to_ci");
}

void ci_rdm12(CiPool* pool, int n, int na, int nb, hipStream_t st, const double* bra, const double* ket, double scale,
              double* gamma, double* Gamma, double* overlap) {
  DMRG_REQUIRE(n >= 1 && n <= 16, ST_EINVAL, "RDMs from CI vectors need 1..16 orbitals");
  const long NA = binom(n, na), NB = binom(n, nb);
  const int n2 = n * n, rows = n2 + 1;
  Work w(pool, n, na, nb, st);
  std::vector<GramRow> list;
  for (int x = 0; x < n2; ++x) list.push_back({0, x, 0});
  list.push_back({0, n2, 0});
  const bool same = bra == ket;
  if (same) gram(w, n, true, bra, list, nullptr, {}, NA, NB, st);
  else gram(w, n, false, bra, list, ket, list, NA, NB, st);
  w->out.reserve((size_t)(n2 + (long)n2 * n2) * 8);
  double *dg = w->out.as<double>(), *dG = dg + n2;
  launch_rdm_assemble(w->G.as<double>(), rows, n, scale, dg, dG, st);
  if (gamma) hip_check(hipMemcpyAsync(gamma, dg, (size_t)n2 * 8, hipMemcpyDeviceToHost, st), "rdm out");
  if (Gamma) hip_check(hipMemcpyAsync(Gamma, dG, (size_t)n2 * n2 * 8, hipMemcpyDeviceToHost, st), "rdm out");
  if (overlap)
    hip_check(hipMemcpyAsync(overlap, w->G.as<double>() + (long)n2 * rows + n2, 8, hipMemcpyDeviceToHost, st), "rdm out");
  hip_check(hipStreamSynchronize(st), "rdm");
}

}  // namespace dmrg
