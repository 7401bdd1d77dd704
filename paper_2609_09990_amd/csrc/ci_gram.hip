// Gram products of excited CI vectors and the two-electron intermediates, with
// the excited copies formed where they are used.
//
// gram: G[i][j] = sum_d A_i[d] B_j[d] over the determinants d, where a row is a CI
// vector or an excited copy E_rs of one (GramRow).  The copies used to be written
// out and read back by a GEMM (5 GB each way for the three-body density at
// CAS(10,10)); here a workgroup takes a range of determinants, 32 at a time,
// gathers its rows' values (two table entries and at most two amplitudes each, of
// vectors that stay in the caches) into LDS and multiplies them on fp64 MFMA,
// keeping its 16 x 16 blocks of G in registers to the end of the range.  The next
// 32 determinants' gathers are in flight during the products.  A group is the
// whole A list with up to 128 B rows; a list of block pairs says which blocks are
// wanted (a symmetric product takes half of them and gathers its rows once).
// Bound by the gathers' instructions and the MFMAs together.  CAS(12,12) 1-/2-RDM:
// 6.5 -> 0.64 ms per call (this kernel 0.57 ms, 32 TFLOP/s of wanted blocks; it was
// two products of 0.94 ms, two passes of copies of 0.24 and 4 ms of host tables and
// allocations); three-body density at CAS(10,10): 76 -> 2.7 ms (2.1 ms here; 9 ms of
// kernels before, the rest the allocation of 4 GB of copies).  Sorting the rows by
// excitation instead of by source vector took 4.2 ms, 64-bit index arithmetic 4.0.
//
// uv: U = F^T (F T) for T_x = E_x c (F the Cholesky factors, nq x n^2), 32
// determinants at a time: T and F T stay in LDS, only U is written.  V c at (6, 5)
// electrons in 12 orbitals with 64 factors: 6.1 -> 1.6 ms (1.4 ms here; two GEMMs
// through memory took 1.1 ms, the copies and the sum 0.7, allocations the rest).
#include <hip/hip_runtime.h>

#include "ci.hpp"

namespace dmrg {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kDet = 32;      // determinants of a slice
constexpr int kDPitch = 34;   // LDS row pitch of a slice: k pairs of 16 rows without bank conflicts
constexpr int kThreads = 512;

// Values of NR rows at determinant d = (ia, ib): (E_x src)[d], with oa = x na + ia
// and ob = x nb + ib the rows' table entries.  Without branches and in stages (all
// table entries, then all amplitudes, then the sums), so that a thread waits for
// two round trips in all instead of four per row; an absent excitation reads the
// determinant itself and drops it.  All offsets are 32-bit.
template <int NR>
__device__ inline void gather_rows(const double* const (&src)[NR], const int (&oa)[NR], const int (&ob)[NR], int d,
                                   int ib, int row0, const int* __restrict__ ta, const int* __restrict__ tb,
                                   double* v) {
  int xa[NR], xb[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    xa[i] = ta[(unsigned)oa[i]];
    xb[i] = tb[(unsigned)ob[i]];
  }
  double a[NR], b[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    a[i] = src[i][(unsigned)(xa[i] ? abs(xa[i]) - 1 + ib : d)];
    b[i] = src[i][(unsigned)(xb[i] ? abs(xb[i]) - 1 + row0 : d)];
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const double s = xa[i] ? (xa[i] > 0 ? a[i] : -a[i]) : 0.0;
    const double t = xb[i] ? (xb[i] > 0 ? b[i] : -b[i]) : 0.0;
    v[i] = s + t;
  }
}

// NBW: blocks per wave; ROWS: rows of A and B (one list when SYM) the LDS holds.
template <int NBW, int ROWS, bool SYM>
__global__ __launch_bounds__(kThreads, NBW <= 7 ? 4 : 2) void gram_kernel(GramArgs P) {
  constexpr int RT = ROWS / 16;                            // rows a thread gathers
  constexpr int BR = RT == 17 ? 6 : 5;                     // rows of a gather stage
  __shared__ __align__(16) double S[ROWS * kDPitch];
  struct Row {  // source vector, table offsets of the excitation
    const double* src;
    int ta, tb;
  };
  __shared__ Row L[ROWS];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kq = lane >> 4;
  const GramGroup g = P.groups[blockIdx.y];
  const int rows = SYM ? P.rows_a : P.rows_a + g.rows_b;
  const int dl = tid & 31, rg = tid >> 5;
  v4d acc[NBW];
  int ao[NBW], bo[NBW];
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    acc[t] = (v4d){0.0, 0.0, 0.0, 0.0};
    const int p = 8 * t + wave;
    const int2 ij = p < g.np ? P.pairs[g.p0 + p] : int2{0, 0};
    ao[t] = __builtin_amdgcn_readfirstlane(ij.x * 16 * kDPitch);
    bo[t] = __builtin_amdgcn_readfirstlane(((SYM ? 0 : P.rows_a) + ij.y * 16) * kDPitch);
  }
  for (int row = tid; row < ROWS; row += kThreads) {
    const bool a = SYM || row < P.rows_a;
    GramRow e{0, P.zero, 0};
    if (row < rows) e = a ? P.list_a[row] : P.list_b[g.b0 + row - P.rows_a];
    L[row] = {(a ? P.src_a : P.src_b) + e.src, e.x * P.na, e.x * P.nb};
  }
  __syncthreads();
  const long nsl = (P.ndet + kDet - 1) / kDet;
  const long c0 = nsl * blockIdx.x / gridDim.x, c1 = nsl * (blockIdx.x + 1) / gridDim.x;
  double v[RT];
  auto gather = [&](long c) {
    const bool in = c * kDet + dl < P.ndet;
    const int d = in ? (int)(c * kDet) + dl : 0;
    const int ia = (int)((unsigned)d / (unsigned)P.nb), row0 = ia * P.nb, ib = d - row0;
#pragma unroll
    for (int i0 = 0; i0 < RT; i0 += BR) {
      const double* src[BR];
      int oa[BR], ob[BR];
#pragma unroll
      for (int i = 0; i < BR; ++i) {
        const Row e = L[min(rg + 16 * (i0 + i), ROWS - 1)];
        src[i] = e.src;
        oa[i] = e.ta + ia;
        ob[i] = e.tb + ib;
      }
      double w[BR];
      gather_rows<BR>(src, oa, ob, d, ib, row0, P.ta, P.tb, w);
#pragma unroll
      for (int i = 0; i < BR; ++i)
        if (i0 + i < RT) v[i0 + i] = in ? w[i] : 0.0;
    }
  };
  if (c0 < c1) gather(c0);
  for (long c = c0; c < c1; ++c) {
    __syncthreads();  // the previous slice is multiplied
#pragma unroll
    for (int i = 0; i < RT; ++i) S[(rg + 16 * i) * kDPitch + dl] = v[i];
    __syncthreads();
    if (c + 1 < c1) gather(c + 1);
#pragma unroll
    for (int kb = 0; kb < kDet / 8; ++kb) {
      const double* s = S + r * kDPitch + 8 * kb + 2 * kq;
#pragma unroll
      for (int t = 0; t < NBW; ++t)
        if (8 * t + wave < g.np) {
          const double2 a = *reinterpret_cast<const double2*>(s + ao[t]);
          const double2 b = *reinterpret_cast<const double2*>(s + bo[t]);
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc[t], 0, 0, 0);
          acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, acc[t], 0, 0, 0);
        }
    }
  }
  // accumulator element q: row kq + 4 q, column r of the block
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int p = 8 * t + wave;
    if (p >= g.np) continue;
    double* o = P.partial + ((long)(g.p0 + p) * gridDim.x + blockIdx.x) * 256;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[(kq + 4 * q) * 16 + r] = acc[t][q];
  }
}

// One workgroup per block of G: its partial blocks in order within 4 interleaved
// groups, then the groups in order.
__global__ __launch_bounds__(1024) void gram_sum_kernel(GramArgs P, int nsplit, int ngroups) {
  __shared__ double sh[3][256];
  const int p = blockIdx.x, e = threadIdx.x & 255, w = threadIdx.x >> 8;
  const double* s = P.partial + (long)p * nsplit * 256 + e;
  double acc = 0.0;
#pragma unroll 8
  for (int x = w; x < nsplit; x += 4) acc += s[(long)x * 256];
  if (w) sh[w - 1][e] = acc;
  __syncthreads();
  if (w) return;
  acc = ((acc + sh[0][e]) + sh[1][e]) + sh[2][e];
  int g = 0;
  while (g + 1 < ngroups && p >= P.groups[g + 1].p0) ++g;
  const int2 ij = P.pairs[p];
  const int i = 16 * ij.x + (e >> 4), j = P.groups[g].b0 + 16 * ij.y + (e & 15);
  if (i >= P.m || j >= P.n) return;
  P.G[(long)i * P.n + j] = acc;
  if (P.sym) P.G[(long)j * P.n + i] = acc;
}

constexpr int kUPitch = 48;  // LDS row pitch: lane groups of 4 rows on different halves of the banks
constexpr int kUQ = 64;      // factors of a pass

// One slice of 32 determinants per workgroup and step: wave w computes block
// (w >> 1, w & 1) of F T (64 x 32 per pass of factors) and blocks w, w + 8, ... of
// U (n^2 x 32).
template <int XB>  // 16-row blocks of the n^2 excitations
__global__ __launch_bounds__(kThreads, 2) void uv_kernel(const double* __restrict__ c, int na, int nb, int n2, int nq,
                                                         const int* __restrict__ ta, const int* __restrict__ tb,
                                                         const double* __restrict__ F, double* __restrict__ U,
                                                         long ndet) {
  constexpr int RT = XB, UB = (2 * XB + 7) / 8;
  __shared__ __align__(16) double T[16 * XB * kUPitch];
  __shared__ __align__(16) double Wq[kUQ * kUPitch];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kq = lane >> 4;
  const int dl = tid & 31, rg = tid >> 5;
  const long nsl = (ndet + kDet - 1) / kDet;
  double v[RT];
  auto gather = [&](long sl) {
    const bool in = sl * kDet + dl < ndet;
    const int d = in ? (int)(sl * kDet) + dl : 0;
    const int ia = (int)((unsigned)d / (unsigned)nb), row0 = ia * nb, ib = d - row0;
    constexpr int BR = XB == 9 ? 9 : 8;
#pragma unroll
    for (int i0 = 0; i0 < RT; i0 += BR) {
      const double* src[BR];
      int oa[BR], ob[BR];
#pragma unroll
      for (int i = 0; i < BR; ++i) {
        const int x = min(rg + 16 * (i0 + i), n2 + 1);  // row n2 + 1 of the tables: none
        src[i] = c;
        oa[i] = (x < n2 ? x : n2 + 1) * na + ia;
        ob[i] = (x < n2 ? x : n2 + 1) * nb + ib;
      }
      gather_rows<BR>(src, oa, ob, d, ib, row0, ta, tb, v + i0);
#pragma unroll
      for (int i = 0; i < BR; ++i) v[i0 + i] = in ? v[i0 + i] : 0.0;
    }
  };
  // this wave's rows of the first pass of factors stay in registers for n <= 12
  constexpr bool KEEP = XB <= 9;
  const int qr0 = 16 * (wave >> 1) + r;
  double fk[KEEP ? 4 * XB : 1];
  if constexpr (KEEP) {
#pragma unroll
    for (int s = 0; s < 4 * XB; ++s) fk[s] = qr0 < nq && 4 * s + kq < n2 ? F[(long)qr0 * n2 + 4 * s + kq] : 0.0;
  }
  if ((long)blockIdx.x < nsl) gather(blockIdx.x);
  for (long sl = blockIdx.x; sl < nsl; sl += gridDim.x) {
    __syncthreads();  // T and Wq of the previous slice are read
#pragma unroll
    for (int i = 0; i < RT; ++i) T[(rg + 16 * i) * kUPitch + dl] = v[i];
    __syncthreads();
    if (sl + gridDim.x < nsl) gather(sl + gridDim.x);
    v4d u[UB];
#pragma unroll
    for (int t = 0; t < UB; ++t) u[t] = (v4d){0.0, 0.0, 0.0, 0.0};
    for (int q0 = 0; q0 < nq; q0 += kUQ) {
      // F T: rows q0 + 16 (wave >> 1) + r, columns 16 (wave & 1) + r
      v4d w = (v4d){0.0, 0.0, 0.0, 0.0};
      const int qr = q0 + 16 * (wave >> 1) + r;
      const double* f = F + (long)(qr < nq ? qr : 0) * n2;
      const double* t0 = T + 16 * (wave & 1) + r;
      if (KEEP && q0 == 0) {
#pragma unroll
        for (int s = 0; s < 4 * XB; ++s)
          w = __builtin_amdgcn_mfma_f64_16x16x4f64(fk[KEEP ? s : 0], t0[(4 * s + kq) * kUPitch], w, 0, 0, 0);
      } else {
        // two chains: behind their loads, one leaves each MFMA waiting for the one before
        // (16 orbitals, 16 factors: 2.95 ms per call against 2.72)
        v4d w2 = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int s = 0; s < 4 * XB; s += 2) {
          const int x = 4 * s + kq;
          const double a = qr < nq && x < n2 ? f[x] : 0.0, a2 = qr < nq && x + 4 < n2 ? f[x + 4] : 0.0;
          w = __builtin_amdgcn_mfma_f64_16x16x4f64(a, t0[x * kUPitch], w, 0, 0, 0);
          w2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a2, t0[(x + 4) * kUPitch], w2, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] += w2[q];
      }
      if (q0 > 0) __syncthreads();  // Wq of the previous pass is read
      // rows past the last factor are zeros, also where T is not finite (0 x inf)
      if (q0 + kUQ > nq) {
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = q0 + 16 * (wave >> 1) + kq + 4 * q < nq ? w[q] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) Wq[(16 * (wave >> 1) + kq + 4 * q) * kUPitch + 16 * (wave & 1) + r] = w[q];
      __syncthreads();
      // U += F^T (F T): rows x, K over this pass's factors
      const int nk = min(kUQ, nq - q0);
#pragma unroll 4
      for (int s = 0; s < (nk + 3) / 4; ++s) {
        const int q = 4 * s + kq;
#pragma unroll
        for (int t = 0; t < UB; ++t) {
          const int b = wave + 8 * t;
          if (b < 2 * XB) {
            const int x = 16 * (b >> 1) + r;
            const double a = q < nk && x < n2 ? F[(long)(q0 + q) * n2 + x] : 0.0;
            u[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Wq[q * kUPitch + 16 * (b & 1) + r], u[t], 0, 0, 0);
          }
        }
      }
    }
#pragma unroll
    for (int t = 0; t < UB; ++t) {
      const int b = wave + 8 * t;
      if (b >= 2 * XB) continue;
      const long d = sl * kDet + 16 * (b & 1) + r;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int x = 16 * (b >> 1) + kq + 4 * q;
        if (x < n2 && d < ndet) U[(long)x * ndet + d] = u[t][q];
      }
    }
  }
}

}  // namespace

void launch_gram(const GramArgs& P, int ngroups, int npairs, int max_pairs, int max_rows, int nsplit, hipStream_t s) {
  if (ngroups <= 0 || npairs <= 0) return;
  const dim3 grid(nsplit, ngroups);
  // the smallest instance that holds the rows and the pairs of every group
  if (P.sym && max_rows <= 160 && max_pairs <= 56) gram_kernel<7, 160, true><<<grid, kThreads, 0, s>>>(P);
  else if (P.sym) gram_kernel<20, 272, true><<<grid, kThreads, 0, s>>>(P);
  else if (max_rows <= 240 && max_pairs <= 56) gram_kernel<7, 240, false><<<grid, kThreads, 0, s>>>(P);
  else if (max_rows <= 272 && max_pairs <= 72) gram_kernel<9, 272, false><<<grid, kThreads, 0, s>>>(P);
  else gram_kernel<17, 400, false><<<grid, kThreads, 0, s>>>(P);
  gram_sum_kernel<<<npairs, 1024, 0, s>>>(P, nsplit, ngroups);
}

void launch_ci_uv(const double* c, int na, int nb, int n2, int nq, const int* ta, const int* tb, const double* F,
                  double* U, long ndet, hipStream_t s) {
  if (ndet <= 0) return;
  const long nsl = (ndet + kDet - 1) / kDet;
  const int grid = (int)(nsl < 512 ? nsl : 512);  // two workgroups per CU
  if (n2 <= 144) uv_kernel<9><<<grid, kThreads, 0, s>>>(c, na, nb, n2, nq, ta, tb, F, U, ndet);
  else uv_kernel<16><<<grid, kThreads, 0, s>>>(c, na, nb, n2, nq, ta, tb, F, U, ndet);
}

}  // namespace dmrg
