// Determinant-space (CI) view of a state and its reduced density matrices: the
// device CI pipeline of the paper's Sec. III (colexicographic string ranks,
// determinant-string enumeration, one- and two-body density matrices formed on
// the device), used here for the 1-/2-RDMs and transition RDMs of MPS states.
//
// Conventions (shared with the integrals of Sec. II.A):
// * E_pq = sum_sigma a+_{p sigma} a_{q sigma}; a determinant is
//   (prod_{p in I_a} a+_{p alpha})(prod_{p in I_b} a+_{p beta})|0>, creators in
//   ascending orbital order, all alpha before all beta;
// * strings are ranked colexicographically, rank = sum_t C(o_t, t + 1) over the
//   sorted occupied orbitals o_0 < o_1 < ...;
// * a CI vector is the row-major matrix c[I_a][I_b] (N_a x N_b).
// The MPS site basis orders spin orbitals 0a, 0b, 1a, 1b, ... (s = n_a + 2 n_b),
// so a site-product amplitude enters c with the sign of moving every alpha
// creator in front of the beta creators of lower orbitals:
// (-1)^{sum over alpha-occupied p of the number of beta electrons below p}.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <memory>
#include <mutex>
#include <vector>

#include "solver.hpp"

namespace dmrg {

// One middle-cut sector of the MPS-to-CI scatter: its prefix x suffix
// amplitude matrix (row-major, n_pre x n_suf, at amp_off) and its rows of the
// prefix / suffix rank and sign tables.
struct CiSector {
  long amp_off;
  long pre_off, suf_off;
  int n_pre, n_suf;
};

// c[(pa + sa) * nb + (pb + sb)] = ps * ss * amp, over every sector's pairs.
void launch_ci_scatter(const double* amp, const CiSector* secs, int n_secs, const int* pa, const int* pb,
                       const double* ps, const int* sa, const int* sb, const double* ss, double* c, long nb,
                       hipStream_t s);

// Excitation tables (N = na nb < 2^31 determinants): for x = r n + s < n2,
// tb[x * nb + J] is +-(I + 1) when E_rs |I> = +-|J> within the beta strings, 0 when
// there is no I; ta[x * na + J] is +-(I nb + 1) likewise (I nb: where alpha string
// I's row starts).  Row n2 is the identity (alpha table: I = J, beta table: none),
// row n2 + 1 holds zeros.
//
// Excited copies of a CI vector: T[x * N + d] = (E_rs c)[d].
void launch_ci_excite(const double* c, long na, long nb, int n2, const int* ta, const int* tb, double* T,
                      hipStream_t s);
// Gram products of excited vectors (ci_gram.hip).  A row: the vector at element
// offset src of its side's base, excited by row x of the tables.
struct GramRow {
  long src;
  int x, pad;
};
// B rows b0 .. b0 + rows_b (a multiple of 16) against every A row; block pairs
// [p0, p0 + np) of the pair table: (A block, B block of the group).
struct GramGroup {
  int b0, rows_b, p0, np;
};
struct GramArgs {
  const double *src_a, *src_b;
  const GramRow *list_a, *list_b;  // padded with zero rows to multiples of 16
  const GramGroup* groups;         // ascending p0, back to back
  const int2* pairs;
  const int *ta, *tb;
  int na, nb;
  long ndet;
  int zero;         // the tables' row of zeros
  int rows_a;       // a multiple of 16
  int m, n;         // rows and columns of G that are wanted
  int sym;          // A and B are one list: pairs of blocks i >= j, G filled both ways
  double* partial;  // npairs x nsplit x 256
  double* G;        // m x n
};
constexpr int kGramRows = 128;  // B rows of a group (one list of up to 272 rows when symmetric)
// max_pairs, max_rows: the largest np and (A and B) rows of a group.
void launch_gram(const GramArgs& P, int ngroups, int npairs, int max_pairs, int max_rows, int nsplit, hipStream_t s);
// U[x * N + d] = sum_Q F[Q][x] sum_y F[Q][y] (E_y c)[d] (F row-major nq x n2).
void launch_ci_uv(const double* c, int na, int nb, int n2, int nq, const int* ta, const int* tb, const double* F,
                  double* U, long ndet, hipStream_t s);
// out[d] = scale * sum_{x < n2} (E_x U_x)[d] over the rows U_x = U + x ldu.
void launch_ci_apply_sum(const double* U, long ldu, long na, long nb, int n2, const int* ta, const int* tb,
                         double scale, double* out, long ndet, hipStream_t s);
// Gamma3[p q r s t u] = scale <E_qp bra | E_rs E_tu ket> from G (n2 rows E_qp bra;
// columns: E_rs E_tu ket for X = rs >= Y = tu at Y n2 - Y (Y - 1) / 2 + X - Y, then E_x ket
// from column n2 (n2 + 1) / 2 on); X < Y by E_rs E_tu = E_tu E_rs + d_st E_ru - d_ru E_ts.
void launch_rdm3_assemble(const double* G, int n, double scale, double* out, hipStream_t s);

// gamma[pq] = scale G[n2][pq]; Gamma[pqrs] = scale (G[qp][rs] - d_qr G[n2][ps])
// with G the (n2 + 1) x (n2 + 1) product of the excited copies (row-major, ldg).
void launch_rdm_assemble(const double* G, int ldg, int n, double scale, double* gamma, double* Gamma,
                         hipStream_t s);

// Device tables and scratch of the determinant-space calls of one problem.  A call
// checks a set out, uses it alone and gives it back with its work done, so calls
// from several threads and streams never share one; at most two idle sets are
// kept, each up to kKeep bytes, until the problem is destroyed or an allocation
// fails.
struct CiWork {
  int device = -1;
  bool tables = false;
  DevMem ta, tb;              // excitation tables
  DevMem T1, T2, part, G, out, lists, F;
  std::vector<DevMem*> scratch() { return {&T1, &T2, &part, &G, &out, &lists, &F}; }
};
class CiPool final : public IdleMemory {
 public:
  CiPool() { enroll(); }
  ~CiPool() { retire(); }
  // holds the largest three-body density: (6, 6) electrons in 12 orbitals, two vectors,
  // 2.15e9 bytes (at 2 GiB every such call freed and allocated one set of copies)
  static constexpr size_t kKeep = size_t(9) << 28;
  std::unique_ptr<CiWork> take();
  void give(std::unique_ptr<CiWork> w);
  void drop() override;

 private:
  std::mutex m_;
  std::vector<std::unique_ptr<CiWork>> idle_;
};

// Two-orbital density matrices of a CI vector (unnormalised), for every pair
// (pairs[2 p], pairs[2 p + 1]), i < j: with the pair's spin orbitals moved to the
// front in the order (i alpha, j alpha, i beta, j beta), rho = sum over the
// configurations of the other orbitals of v v^T.  Only the 36 entries of the 9
// blocks of equal pair (N_alpha, N_beta) can be non-zero; partial[(p * nblk + b)
// * 36 + e] receives workgroup b's sums (nblk = grid size per pair), and
// launch_orb_sum adds them in order into out[p * 36 + e].  sa / sb: the strings
// by rank; rank_a / rank_b: the rank of every n-bit mask (-1 if not a string).
void launch_orb_pairs(const double* c, const uint32_t* sa, const uint32_t* sb, const int* rank_a, const int* rank_b,
                      long nb, long ndet, const int* pairs, int npairs, int nblk, double* partial, hipStream_t s);
void launch_orb_sum(const double* partial, int npairs, int nblk, double* out, hipStream_t s);

}  // namespace dmrg
