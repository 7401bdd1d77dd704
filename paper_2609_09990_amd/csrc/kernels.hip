// gfx950 kernels for the two-site sigma path.
//
// The workhorse is a grouped block GEMM: every output tile of sigma (or of a
// new environment, or of an intermediate T = X psi) accumulates its block
// products ("items") in a fixed order with MFMA, so results are bitwise
// reproducible (no atomics; split-K partial tiles are summed in order by
// splitk_reduce).  Sigma takes the slab kernel (phase A, gemm_slab.hip) and the
// stream kernel (phase B, gemm_stream.hip) in every precision, the gradient's
// G = P Q^T the stream kernel; here:
//  * w32_tile: one wave per (16 RB) x (16 CB) tile reading operands straight
//    from memory (fp64: environment updates, the gradient's row products);
//  * gemm_f64 / gemm_f32 / gemm_bf16: plain 64 x 64 LDS tiles, four waves of
//    32 x 32 (one-off products: two-site forms, overlaps, projections, the hidden
//    layer of few rows, dmrg_block_gemm).
// Plus the Davidson BLAS-1 kernels, the one-workgroup Jacobi eigensolver, the
// diagonal, premix / pairmix and precision conversions.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <stdexcept>

#include "bf16.hpp"
#include "jacobi.hpp"
#include "kernels.hpp"

namespace dmrg {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));

namespace {

constexpr int TM = 64, TN = 64, TK = 16, LDP = TM + 2;

__device__ inline float to_f(float x) { return x; }
__device__ inline float to_f(double x) { return (float)x; }
__device__ inline float to_f(uint16_t x) { return __uint_as_float(((uint32_t)x) << 16); }
__device__ inline double to_d(double x) { return x; }
__device__ inline double to_d(float x) { return (double)x; }
// Loads a 64 x 16 A tile (k-major into LDS) and a 16 x 64 B tile, scaling A by coef.
template <int MODE, typename TA, typename TB, typename TS>
__device__ inline void load_tiles(TS (*As)[LDP], TS (*Bs)[LDP], const TA* A, const TB* B, int lda,
                                  int ldb, int K, int k0, int m0, int M, int n0, int N,
                                  double coef, int tid) {
  if (MODE == GEMM_NN || MODE == GEMM_NT) {
    int m = tid >> 2, kq = (tid & 3) * 4;
    int gm = m0 + m;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int k = kq + j;
      double v = 0.0;
      if (gm < M && k0 + k < K) v = to_d(A[(long)gm * lda + k0 + k]) * coef;
      As[k][m] = (TS)v;
    }
  } else {
    int k = tid >> 4, mq = (tid & 15) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int m = mq + j;
      double v = 0.0;
      if (m0 + m < M && k0 + k < K) v = to_d(A[(long)(k0 + k) * lda + m0 + m]) * coef;
      As[k][m] = (TS)v;
    }
  }
  if (MODE == GEMM_NN || MODE == GEMM_TN) {
    int k = tid >> 4, nq = (tid & 15) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int n = nq + j;
      TS v = (TS)0;
      if (n0 + n < N && k0 + k < K) v = (TS)to_d(B[(long)(k0 + k) * ldb + n0 + n]);
      Bs[k][n] = v;
    }
  } else {
    int n = tid >> 2, kq = (tid & 3) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int k = kq + j;
      TS v = (TS)0;
      if (n0 + n < N && k0 + k < K) v = (TS)to_d(B[(long)(n0 + n) * ldb + k0 + k]);
      Bs[k][n] = v;
    }
  }
}

template <int MODE>
__global__ __launch_bounds__(256) void gemm_f64(const GemmUnit* __restrict__ units,
                                                const GemmItem* __restrict__ items) {
  __shared__ double As[TK][LDP];
  __shared__ double Bs[TK][LDP];
  const GemmUnit u = units[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  v4d acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};
  for (int it = u.ib; it < u.ie; ++it) {
    const GemmItem g = items[it];
    const double* A = (const double*)g.A;
    const double* B = (const double*)g.B;
    for (int k0 = 0; k0 < g.K; k0 += TK) {
      load_tiles<MODE, double, double, double>(As, Bs, A, B, g.lda, g.ldb, g.K, k0, u.m0, u.M,
                                               u.n0, u.N, g.coef, tid);
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < TK; kk += 4) {
        double a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = As[kk + (lane >> 4)][wr + 16 * i + (lane & 15)];
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = Bs[kk + (lane >> 4)][wc + 16 * j + (lane & 15)];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      __syncthreads();
    }
  }
  double* C = (double*)u.C;
  // v_mfma_f64_16x16x4f64 accumulator: lane l, element r holds row l/16 + 4r,
  // column l%16 (measured; the f32/bf16 16x16 ops hold row 4(l/16) + r instead)
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int gm = u.m0 + wr + 16 * i + (lane >> 4) + 4 * r;
        int gn = u.n0 + wc + 16 * j + (lane & 15);
        if (gm < u.M && gn < u.N) {
          long idx = (long)gm * u.ldc + gn;
          double v = acc[i][j][r];
          C[idx] = u.accumulate ? C[idx] + v : v;
        }
      }
}

template <int MODE, typename TA, typename TB>
__global__ __launch_bounds__(256) void gemm_f32(const GemmUnit* __restrict__ units,
                                                const GemmItem* __restrict__ items) {
  __shared__ float As[TK][LDP];
  __shared__ float Bs[TK][LDP];
  const GemmUnit u = units[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  for (int it = u.ib; it < u.ie; ++it) {
    const GemmItem g = items[it];
    for (int k0 = 0; k0 < g.K; k0 += TK) {
      load_tiles<MODE, TA, TB, float>(As, Bs, (const TA*)g.A, (const TB*)g.B, g.lda, g.ldb, g.K,
                                      k0, u.m0, u.M, u.n0, u.N, g.coef, tid);
      __syncthreads();
#pragma unroll
      for (int kk = 0; kk < TK; kk += 4) {
        float a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = As[kk + (lane >> 4)][wr + 16 * i + (lane & 15)];
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = Bs[kk + (lane >> 4)][wc + 16 * j + (lane & 15)];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      __syncthreads();
    }
  }
  float* C = (float*)u.C;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int gm = u.m0 + wr + 16 * i + 4 * (lane >> 4) + r;
        int gn = u.n0 + wc + 16 * j + (lane & 15);
        if (gm < u.M && gn < u.N) {
          long idx = (long)gm * u.ldc + gn;
          float v = acc[i][j][r];
          C[idx] = u.accumulate ? C[idx] + v : v;
        }
      }
}

// bf16 operands, fp32 accumulation (A times the item's coefficient is rounded to bf16
// in LDS).  One v_mfma_f32_16x16x16_bf16 per 16-deep k tile.
template <int MODE>
__global__ __launch_bounds__(256) void gemm_bf16(const GemmUnit* __restrict__ units,
                                                 const GemmItem* __restrict__ items) {
  __shared__ uint16_t As[TK][LDP];
  __shared__ uint16_t Bs[TK][LDP];
  const GemmUnit u = units[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  for (int it = u.ib; it < u.ie; ++it) {
    const GemmItem g = items[it];
    const uint16_t* A = (const uint16_t*)g.A;
    const uint16_t* B = (const uint16_t*)g.B;
    const float coef = (float)g.coef;
    for (int k0 = 0; k0 < g.K; k0 += TK) {
      if (MODE == GEMM_NN || MODE == GEMM_NT) {
        int m = tid >> 2, kq = (tid & 3) * 4;
        int gm = u.m0 + m;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int k = kq + j;
          float v = 0.f;
          if (gm < u.M && k0 + k < g.K) v = to_f(A[(long)gm * g.lda + k0 + k]) * coef;
          As[k][m] = f2bf(v);
        }
      } else {
        int k = tid >> 4, mq = (tid & 15) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int m = mq + j;
          float v = 0.f;
          if (u.m0 + m < u.M && k0 + k < g.K) v = to_f(A[(long)(k0 + k) * g.lda + u.m0 + m]) * coef;
          As[k][m] = f2bf(v);
        }
      }
      if (MODE == GEMM_NN || MODE == GEMM_TN) {
        int k = tid >> 4, nq = (tid & 15) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int n = nq + j;
          uint16_t v = 0;
          if (u.n0 + n < u.N && k0 + k < g.K) v = B[(long)(k0 + k) * g.ldb + u.n0 + n];
          Bs[k][n] = v;
        }
      } else {
        int n = tid >> 2, kq = (tid & 3) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int k = kq + j;
          uint16_t v = 0;
          if (u.n0 + n < u.N && k0 + k < g.K) v = B[(long)(u.n0 + n) * g.ldb + k0 + k];
          Bs[k][n] = v;
        }
      }
      __syncthreads();
      v4s a[2], b[2];
      const int kb = 4 * (lane >> 4);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) a[i][q] = (short)As[kb + q][wr + 16 * i + (lane & 15)];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) b[j][q] = (short)Bs[kb + q][wc + 16 * j + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[j], acc[i][j], 0, 0, 0);
      __syncthreads();
    }
  }
  float* C = (float*)u.C;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int gm = u.m0 + wr + 16 * i + 4 * (lane >> 4) + r;
        int gn = u.n0 + wc + 16 * j + (lane & 15);
        if (gm < u.M && gn < u.N) {
          long idx = (long)gm * u.ldc + gn;
          float v = acc[i][j][r];
          C[idx] = u.accumulate ? C[idx] + v : v;
        }
      }
}

// Small-tile fp64 GEMM: one wave owns a 32x32 tile (2x2 MFMA 16x16 blocks) and
// loads its MFMA operands straight from global memory (k step 4, no LDS, no
// barriers), so short-K items cost little padding and waves never wait on each
// other.  Four independent waves per workgroup.  accumulate == 2 writes the
// tile into a 32x32 partial slot (split-K), reduced later in a fixed order.
template <int MODE>
__device__ inline double ld_a(const double* A, int lda, int m, int k) {
  return MODE == GEMM_TN ? A[(long)k * lda + m] : A[(long)m * lda + k];
}
template <int MODE>
__device__ inline double ld_b(const double* B, int ldb, int k, int n) {
  return MODE == GEMM_NT ? B[(long)n * ldb + k] : B[(long)k * ldb + n];
}

// Two consecutive doubles p[k], p[k+1] of a row (zero past K or for a masked
// row); a full pair is one 16-byte load (8-byte aligned).
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
typedef __attribute__((address_space(1))) const d2u gd2u;      // global memory
typedef __attribute__((address_space(1))) const double gdbl;
__device__ inline void ld_pair(const double* p, int k, int K, bool rowv, double* x) {
  if (rowv && k + 1 < K) {
    const d2u v = *(gd2u*)(p + k);
    x[0] = v.x;
    x[1] = v.y;
  } else {
    x[0] = (rowv && k < K) ? *(gdbl*)(p + k) : 0.0;
    x[1] = 0.0;
  }
}

// Raw buffer loads: a resource covers one operand's extent, loads past it return
// zeros (no fault), so masked lanes need no branches.  Word 3 is the gfx9 raw
// buffer format.
typedef unsigned int v4u32 __attribute__((ext_vector_type(4)));
typedef unsigned int v2u32 __attribute__((ext_vector_type(2)));
constexpr int kBufWord3 = 0x00020000;
__device__ inline __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, kBufWord3);
}
__device__ inline void buf_pair(__amdgpu_buffer_rsrc_t r, int e, double* x) {
  const v4u32 v = __builtin_amdgcn_raw_buffer_load_b128(r, e * 8, 0, 0);
  __builtin_memcpy(&x[0], &v, 8);
  __builtin_memcpy(&x[1], reinterpret_cast<const char*>(&v) + 8, 8);
}
__device__ inline double buf_one(__amdgpu_buffer_rsrc_t r, int e) {
  const v2u32 v = __builtin_amdgcn_raw_buffer_load_b64(r, e * 8, 0, 0);
  double x;
  __builtin_memcpy(&x, &v, 8);
  return x;
}

// One wave computes a (16 RB) x (16 CB) tile: RB x CB fp64 16x16x4 MFMA blocks.
// BUF: every item is known (checked on the host) to fit the buffer-load path, so
// the kernel holds that path alone; otherwise the plain-load paths.  Keeping the
// two apart lets one set of accumulators serve the whole kernel.
template <int MODE, int RB, int CB, bool BUF>
__device__ inline void w32_tile(const GemmUnit& u, const GemmItem* __restrict__ items, int lane) {
  const int r = lane & 15, kq = lane >> 4;
  int am[RB], bn[CB];
  bool av[RB], bv[CB];
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    am[i] = u.m0 + 16 * i + r;
    av[i] = am[i] < u.M;
  }
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    bn[j] = u.n0 + 16 * j + r;
    bv[j] = bn[j] < u.N;
  }
  v4d acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};
  // the next item's descriptor is fetched while the current item computes
  GemmItem gnext;
  if (u.ib < u.ie) gnext = items[u.ib];
  for (int it = u.ib; it < u.ie; ++it) {
    const GemmItem g = gnext;
    if (it + 1 < u.ie) gnext = items[it + 1];
    const double* A = (const double*)g.A;
    const double* B = (const double*)g.B;
    const double c = g.coef;
    // elements of A and B the unit can touch (row-major, leading dims lda, ldb)
    const long ea = (long)(u.M - 1) * g.lda + g.K;
    const long eb = MODE == GEMM_NT ? (long)(u.N - 1) * g.ldb + g.K : (long)(g.K - 1) * g.ldb + u.N;
    if constexpr (BUF) {
      // Same k pairing as below, through buffer loads: a masked row starts past
      // the extent (its loads read zeros), a k past K is zeroed by a select.
      const __amdgpu_buffer_rsrc_t ra = buf_rsrc(A, ea * 8), rb = buf_rsrc(B, eb * 8);
      int ao[RB], bo[CB];
#pragma unroll
      for (int i = 0; i < RB; ++i) ao[i] = av[i] ? am[i] * g.lda : (int)ea;
#pragma unroll
      for (int j = 0; j < CB; ++j) bo[j] = MODE == GEMM_NT ? (bv[j] ? bn[j] * g.ldb : (int)eb) : bn[j];
      const int kfull = g.K - (g.K & 7) + ((g.K & 7) > 4 ? 8 : 0);  // paired blocks; a tail of <= 4 goes alone
      // raw loads of block k0 (masking applied at use), so block k0+8 can be in
      // flight while block k0 is multiplied
      double ta[RB][2], tb[CB][2];
      auto raw = [&](int k0, double (&xa)[RB][2], double (&xb)[CB][2]) {
        const int kk = k0 + 2 * kq;
#pragma unroll
        for (int i = 0; i < RB; ++i) buf_pair(ra, ao[i] + kk, xa[i]);
        if constexpr (MODE == GEMM_NT) {
#pragma unroll
          for (int j = 0; j < CB; ++j) buf_pair(rb, bo[j] + kk, xb[j]);
        } else {
#pragma unroll
          for (int j = 0; j < CB; ++j) {
            xb[j][0] = buf_one(rb, kk * g.ldb + bo[j]);
            xb[j][1] = buf_one(rb, (kk + 1) * g.ldb + bo[j]);
          }
        }
      };
      if (kfull > 0) raw(0, ta, tb);
      for (int k0 = 0; k0 < kfull; k0 += 8) {
        double na[RB][2], nb[CB][2];
        if (k0 + 8 < kfull) raw(k0 + 8, na, nb);
        const int kk = k0 + 2 * kq;
        const bool k0v = kk < g.K, k1v = kk + 1 < g.K;
        double a[RB][2], b[CB][2];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          a[i][0] = k0v ? ta[i][0] * c : 0.0;
          a[i][1] = k1v ? ta[i][1] * c : 0.0;
        }
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          b[j][0] = ((MODE == GEMM_NT || bv[j]) && k0v) ? tb[j][0] : 0.0;
          b[j][1] = ((MODE == GEMM_NT || bv[j]) && k1v) ? tb[j][1] : 0.0;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][h], b[j][h], acc[i][j], 0, 0, 0);
        if (k0 + 8 < kfull) {
#pragma unroll
          for (int i = 0; i < RB; ++i) {
            ta[i][0] = na[i][0];
            ta[i][1] = na[i][1];
          }
#pragma unroll
          for (int j = 0; j < CB; ++j) {
            tb[j][0] = nb[j][0];
            tb[j][1] = nb[j][1];
          }
        }
      }
      if (kfull < g.K) {  // last 1..4 k: one MFMA step, lane kq takes k = kfull + kq
        const int kk = kfull + kq;
        const bool kv = kk < g.K;
        double a[RB], b[CB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          const double t = buf_one(ra, ao[i] + kk);
          a[i] = kv ? t * c : 0.0;
        }
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          const double t = MODE == GEMM_NT ? buf_one(rb, bo[j] + kk) : buf_one(rb, kk * g.ldb + bo[j]);
          b[j] = (kv && (MODE == GEMM_NT || bv[j])) ? t : 0.0;
        }
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int j = 0; j < CB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
      }
    } else if constexpr (MODE == GEMM_NT || MODE == GEMM_NN) {
      (void)ea;
      (void)eb;
      // A runs along k in memory: lane (r, kq) loads the pair k0+2kq, k0+2kq+1 of
      // its rows with one 16-byte load, and the two MFMA steps of an 8-deep block
      // take the even and the odd k of the pairs (the same k order for B, so the
      // product is unchanged).  In NT mode B runs along k too; in NN mode its rows
      // kk and kk+1 are contiguous in n.
      const double* pa[RB];
      const double* pb[CB];
#pragma unroll
      for (int i = 0; i < RB; ++i) pa[i] = A + (long)(av[i] ? am[i] : 0) * g.lda;
#pragma unroll
      for (int j = 0; j < CB; ++j) pb[j] = B + (long)(bv[j] ? bn[j] : 0) * g.ldb;
      for (int k0 = 0; k0 < g.K; k0 += 8) {
        const int kk = k0 + 2 * kq;
        double a[RB][2], b[CB][2];
#pragma unroll
        for (int i = 0; i < RB; ++i) ld_pair(pa[i], kk, g.K, av[i], a[i]);
        if constexpr (MODE == GEMM_NT) {
#pragma unroll
          for (int j = 0; j < CB; ++j) ld_pair(pb[j], kk, g.K, bv[j], b[j]);
        } else {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const bool kv = kk + h < g.K;
            const gdbl* brow = (const gdbl*)(B + (long)(kv ? kk + h : 0) * g.ldb);
#pragma unroll
            for (int j = 0; j < CB; ++j) b[j][h] = (bv[j] && kv) ? brow[bn[j]] : 0.0;
          }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < RB; ++i) {
            const double x = a[i][h] * c;
#pragma unroll
            for (int j = 0; j < CB; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b[j][h], acc[i][j], 0, 0, 0);
          }
      }
    } else {
      for (int k0 = 0; k0 < g.K; k0 += 4) {
        const int ka = k0 + kq;
        const bool kv = ka < g.K;
        double a[RB], b[CB];
#pragma unroll
        for (int i = 0; i < RB; ++i) a[i] = (av[i] && kv) ? ld_a<MODE>(A, g.lda, am[i], ka) * c : 0.0;
#pragma unroll
        for (int j = 0; j < CB; ++j) b[j] = (bv[j] && kv) ? ld_b<MODE>(B, g.ldb, ka, bn[j]) : 0.0;
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int j = 0; j < CB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
      }
    }
  }
  double* C = (double*)u.C;
  // accumulator element q of lane l: row l/16 + 4q, column l%16 (fp64 16x16x4 layout)
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        int tr = 16 * i + kq + 4 * q, tc = 16 * j + r;
        int gm = u.m0 + tr, gn = u.n0 + tc;
        double v = acc[i][j][q];
        if (u.accumulate == 2) {
          C[tr * (16 * CB) + tc] = v;  // partial slot, full tile (masked entries are zero)
        } else if (gm < u.M && gn < u.N) {
          long idx = (long)gm * u.ldc + gn;
          C[idx] = u.accumulate ? C[idx] + v : v;
        }
      }
}

template <int MODE, bool BUF>
__global__ __launch_bounds__(256) void gemm_f64_w32(const GemmUnit* __restrict__ units,
                                                    const GemmItem* __restrict__ items, int n_units) {
  // the wave index is uniform across the wave; saying so keeps the unit and item
  // descriptors (and the buffer resources built from them) in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // NN launches (a factor or environment block feeds every column tile of its
  // unit) give each XCD a contiguous range of units, so a block is fetched into
  // one XCD's L2; workgroups are dispatched to the 8 XCDs round-robin.  NT
  // launches keep the plain order.
  int wg = blockIdx.x;
  if constexpr (MODE == GEMM_NN) {
    const int nb = gridDim.x, q = nb >> 3, rem = nb & 7, x = wg & 7;
    wg = x * q + min(x, rem) + (wg >> 3);
  }
  const int ui = wg * 4 + wave;
  if (ui >= n_units) return;  // whole wave exits; the kernel has no barriers
  const GemmUnit u = units[ui];
  switch (u.shape) {  // 8 * RB + CB: tile (16 RB) x (16 CB)
    case 9: w32_tile<MODE, 1, 1, BUF>(u, items, lane); break;
    case 10: w32_tile<MODE, 1, 2, BUF>(u, items, lane); break;
    case 17: w32_tile<MODE, 2, 1, BUF>(u, items, lane); break;
    case 25: w32_tile<MODE, 3, 1, BUF>(u, items, lane); break;
    case 26: w32_tile<MODE, 3, 2, BUF>(u, items, lane); break;
    case 33: w32_tile<MODE, 4, 1, BUF>(u, items, lane); break;
    case 34: w32_tile<MODE, 4, 2, BUF>(u, items, lane); break;
    default: w32_tile<MODE, 2, 2, BUF>(u, items, lane); break;
  }
}

// One thread per unit.  Planned on the host, the gradient's 330 thousand row
// products at CAS(12,12), M = 256 took 40 ms to list, check and upload against 7 ms
// of kernels; their tables (channel classes x blocks) are a few thousand entries.
// Energy and gradient of a given MPS there: 106 -> 25 ms (with the classes of a
// site in one launch and the long-K product on the stream kernel).
__global__ void grad_expand_kernel(GradView v, int left, const double* env, const double* site, double* out,
                                   GemmUnit* __restrict__ units, GemmItem* __restrict__ items) {
  for (long u = (long)blockIdx.x * blockDim.x + threadIdx.x; u < v.units; u += (long)gridDim.x * blockDim.x) {
    int a = 0, b = v.n_jobs - 1;  // the last job with u0 <= u
    while (a < b) {
      const int m = (a + b + 1) / 2;
      if (v.jobs[m].u0 <= u) a = m;
      else b = m - 1;
    }
    const GradJob J = v.jobs[a];
    const long r = (u - J.u0) / J.ntile;
    const GradTile t = v.tiles[J.tile0 + (u - J.u0 - r * J.ntile)];
    const GradBlock bk = v.blocks[J.blk0 + t.block];
    const GradRow row = v.rows[J.row0 + r];
    const GradSrc x = v.srcs[J.src0 + (long)row.kind * J.nblk + t.block];
    const double *e = env + row.chan + x.env, *s = site + x.site;
    items[u] = {left ? e : s, left ? s : e, x.lda, x.ldb, x.K, 0, 1.0};
    units[u] = {out + J.out + r * J.K + bk.off, bk.mj, bk.mi, bk.mj, t.m0, t.n0, (int)u, (int)u + x.valid, 0, t.shape};
  }
}

__global__ void splitk_reduce_f32(const SplitTile* __restrict__ tiles, const float* __restrict__ slots) {
  // workgroup (tile, chunk of 256 elements): one element per thread
  const SplitTile t = tiles[blockIdx.x];
  const int e = blockIdx.y * blockDim.x + threadIdx.x;
  if (e >= t.tm * t.tn) return;
  const int tr = e / t.tn, tc = e - tr * t.tn;
  const int gm = t.m0 + tr, gn = t.n0 + tc;
  if (gm >= t.M || gn >= t.N) return;
  float acc = 0.f;
  const long step = (long)t.tm * t.tn;
  for (int s = 0; s < t.ns; ++s) acc += slots[t.s0 + s * step + e];
  float* c = (float*)t.C + (long)gm * t.ldc + gn;
  *c = t.acc ? *c + acc : acc;
}

// Split-K reduction: out tile = (out tile if acc) + sum of its partial slots in order.
__global__ void splitk_reduce(const SplitTile* __restrict__ tiles, const double* __restrict__ slots) {
  // workgroup (tile, chunk of 256 elements): one element per thread
  const SplitTile t = tiles[blockIdx.x];
  const int e = blockIdx.y * blockDim.x + threadIdx.x;
  if (e >= t.tm * t.tn) return;
  const int tr = e / t.tn, tc = e - tr * t.tn;
  const int gm = t.m0 + tr, gn = t.n0 + tc;
  if (gm >= t.M || gn >= t.N) return;
  double acc = 0.0;
  const long step = (long)t.tm * t.tn;
  for (int s = 0; s < t.ns; ++s) acc += slots[t.s0 + s * step + e];
  double* c = (double*)t.C + (long)gm * t.ldc + gn;
  *c = t.acc ? *c + acc : acc;
}

__global__ void premix_kernel(double* __restrict__ out, const double* const* __restrict__ srcs,
                              const int* __restrict__ ptr, const double* __restrict__ coef,
                              long nnz) {
  const int f = blockIdx.y;
  const int b = ptr[f], e = ptr[f + 1];
  for (long j = (long)blockIdx.x * blockDim.x + threadIdx.x; j < nnz;
       j += (long)gridDim.x * blockDim.x) {
    double acc = 0.0;
    for (int i = b; i < e; ++i) acc += coef[i] * srcs[i][j];
    out[(long)f * nnz + j] = acc;
  }
}

// out[out_off[g] + j] = sum_{i in [ptr[g], ptr[g+1])} coef[i] * srcs[i][j], j < nnz[g];
// one workgroup per group, sources summed in order.
__global__ void pairmix_kernel(double* __restrict__ out, const double* const* __restrict__ srcs,
                               const int* __restrict__ ptr, const double* __restrict__ coef,
                               const long* __restrict__ out_off, const int* __restrict__ nnz) {
  const int g = blockIdx.x;
  const int b = ptr[g], e = ptr[g + 1], n = nnz[g];
  double* o = out + out_off[g];
  for (int j = threadIdx.x; j < n; j += blockDim.x) {
    double acc = 0.0;
    for (int i = b; i < e; ++i) acc += coef[i] * srcs[i][j];
    o[j] = acc;
  }
}

__global__ void fill_kernel(double* x, long n, double v) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    x[i] = v;
}

__global__ void copy_blocks_kernel(const int64_t* __restrict__ desc, const double* __restrict__ src,
                                   double* __restrict__ dst) {
  const int64_t* d = desc + 9 * blockIdx.x;
  const long so = d[0], srs = d[1], scs = d[2], dof = d[3], drs = d[4], dcs = d[5];
  const int rows = (int)d[6], cols = (int)d[7];
  const double sc = __longlong_as_double((long long)d[8]);
  for (int e = threadIdx.x; e < rows * cols; e += blockDim.x) {
    int r = e / cols, c = e % cols;
    dst[dof + (long)r * drs + (long)c * dcs] = sc * src[so + (long)r * srs + (long)c * scs];
  }
}

__global__ void axpy_dev_kernel(double* __restrict__ y, const double* __restrict__ x,
                                const double* __restrict__ a, double sign, long n) {
  const double s = sign * a[0];
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] += s * x[i];
}

__global__ void copy_kernel(double* __restrict__ dst, const double* __restrict__ src, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

__global__ void fill_f32_kernel(float* x, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    x[i] = 0.f;
}

__global__ void dots_partial(const double* __restrict__ V, long ldv, const double* __restrict__ x,
                             long n, long chunk, double* __restrict__ partial) {
  const int c = blockIdx.x, i = blockIdx.y;
  const long b = (long)c * chunk, e = min(n, b + chunk);
  const double* v = V + (long)i * ldv;
  double acc = 0.0;
  for (long j = b + threadIdx.x; j < e; j += blockDim.x) acc += v[j] * x[j];
  __shared__ double red[256];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[(long)i * gridDim.x + c] = red[0];
}

__global__ void dots_final(const double* __restrict__ partial, int nchunk, double* __restrict__ out) {
  const int i = blockIdx.x;
  __shared__ double red[256];
  double acc = 0.0;
  for (int c = threadIdx.x; c < nchunk; c += blockDim.x) acc += partial[(long)i * nchunk + c];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[i] = red[0];
}

// dots of short vectors in one launch (one workgroup per vector): n <= kDotsOne
// elements take less time than the second launch of the two-pass form.
constexpr long kDotsOne = 16384;
__global__ __launch_bounds__(512) void dots_one(const double* __restrict__ V, long ldv, const double* __restrict__ x,
                                                long n, double* __restrict__ out) {
  const double* v = V + (long)blockIdx.x * ldv;
  double acc = 0.0;
#pragma unroll 4
  for (long j = threadIdx.x; j < n; j += 512) acc += v[j] * x[j];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  __shared__ double red[8];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = red[0];
    for (int w = 1; w < 8; ++w) s += red[w];
    out[blockIdx.x] = s;
  }
}

__global__ void gemv_kernel(const double* __restrict__ V, long ldv, int k,
                            const double* __restrict__ coef, double alpha, double* __restrict__ out,
                            double beta, long n) {
  __shared__ double cs[128];
  for (int i = threadIdx.x; i < k; i += blockDim.x) cs[i] = coef[i];
  __syncthreads();
  for (long j = (long)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (long)gridDim.x * blockDim.x) {
    double acc = 0.0;
    for (int i = 0; i < k; ++i) acc += cs[i] * V[(long)i * ldv + j];
    out[j] = (beta == 0.0 ? 0.0 : beta * out[j]) + alpha * acc;
  }
}

__global__ void scale_by_norm_kernel(double* x, long n, const double* nrm2) {
  const double s = 1.0 / sqrt(nrm2[0]);
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    x[i] *= s;
}

__global__ void precond_diag_kernel(const double* __restrict__ r, const double* __restrict__ d,
                                    const double* __restrict__ theta, double* __restrict__ out, long n) {
  const double th = theta[0];
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    double den = th - d[i];
    if (fabs(den) < 1e-8) den = den < 0 ? -1e-8 : 1e-8;
    out[i] = r[i] / den;
  }
}

// Low-precision copy entries recomputed from fp64 with a shift:
// dst[idx[i]] = round(src[idx[i]] - w[i] * s) (fp32 or bf16 by `bf16`).
__global__ void shift_entries_kernel(const double* __restrict__ src, void* __restrict__ dst, int bf16,
                                     const long* __restrict__ idx, const double* __restrict__ w, long n, double s) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const long e = idx[i];
    const float v = (float)(src[e] - w[i] * s);
    if (bf16) ((uint16_t*)dst)[e] = f2bf(v);
    else ((float*)dst)[e] = v;
  }
}

__global__ void axpy_ratio_kernel(double* __restrict__ y, const double* __restrict__ x, const double* __restrict__ num,
                                  const double* __restrict__ den, double sign, long n) {
  const double a = sign * num[0] / den[0];
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] += a * x[i];
}

__global__ void xpby_ratio_kernel(double* __restrict__ p, const double* __restrict__ z, const double* __restrict__ num,
                                  const double* __restrict__ den, long n) {
  const double b = num[0] / den[0];
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    p[i] = z[i] + b * p[i];
}

__global__ void axpy_kernel(double* __restrict__ y, const double* __restrict__ x, double a, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] += a * x[i];
}

// d[i] += sum_{j<k} V[j ldv + i]^2 (diagonal of a rank-k update V V^T).
__global__ void add_squares_kernel(double* __restrict__ d, const double* __restrict__ V, long ldv, int k, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    double acc = d[i];
    for (int j = 0; j < k; ++j) {
      const double v = V[(long)j * ldv + i];
      acc = fma(v, v, acc);
    }
    d[i] = acc;
  }
}

// Symmetric eigensolver for k <= 64 in one workgroup: cyclic Jacobi with the
// round-robin (circle) pairing, so each round rotates the n/2 disjoint pairs
// (p, q) together (n = k rounded up to even; a pair holding the padding index
// is not rotated).  A pair is rotated when its coupling is significant against
// its diagonal entries.  A round maps each 2 x 2 block of A (rows of pair a,
// columns of pair b) to R_a^T A_ab R_b and each block of V to V_ab R_b; every
// thread derives the angles of its blocks' two pairs from the round's input A
// and writes the other copy of A and V, so a round has one barrier.  Per
// element this is the arithmetic of rotating all rows, then all columns.  The
// iteration ends when no pair is significant (a sweep would rotate nothing) or
// the off-diagonal part is at the rounding level.
__device__ inline void jacobi_pair(int round, int t, int n, int& p, int& q) {
  int x, y;  // 0 <= round, t < n - 1
  if (t == 0) {
    x = round;
    y = n - 1;
  } else {
    x = round + t;
    if (x >= n - 1) x -= n - 1;
    y = round - t;
    if (y < 0) y += n - 1;
  }
  p = min(x, y);
  q = max(x, y);
}
__device__ inline bool jacobi_significant(double apq, double app, double aqq) {
  return fabs(apq) > 1e-300 && fabs(apq) > 1e-15 * __builtin_amdgcn_sqrt(fabs(app * aqq));
}
// rotation of pair (p, q), p < q < k: c = 1, s = 0 when the coupling is not
// significant
struct HwEstimate {
  __device__ static double rsq(double x) { return __builtin_amdgcn_rsq(x); }
  __device__ static double rcp(double x) { return __builtin_amdgcn_rcp(x); }
};
__device__ inline void jacobi_angle(const double (*A)[65], int p, int q, double& c, double& s) {
  const double apq = A[p][q], app = A[p][p], aqq = A[q][q];
  const bool rot = jacobi_significant(apq, app, aqq);
  double cc, ss;
  jacobi_rotation<HwEstimate>(app, aqq, apq, cc, ss);
  c = rot ? cc : 1.0;
  s = rot ? ss : 0.0;
}

__global__ __launch_bounds__(256) void jacobi_eig_kernel(const double* __restrict__ G, int ldg, int k,
                                                         double* __restrict__ evals,
                                                         double* __restrict__ evecs) {
  __shared__ double A[2][64][65];
  __shared__ double V[2][64][65];
  __shared__ double red[2][3][4];
  __shared__ int order[64];
  const int t = threadIdx.x;
  for (int e = t; e < k * k; e += blockDim.x) {  // lower triangle holds the matrix
    const int i = e / k, j = e % k;
    A[0][i][j] = i >= j ? G[(long)i * ldg + j] : G[(long)j * ldg + i];
    V[0][i][j] = (i == j) ? 1.0 : 0.0;
  }
  __syncthreads();
  const int n = k + (k & 1);
  const int half = n / 2;
  int ba[4], bb[4];  // this thread's blocks of a round
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = t + 256 * i;
    ba[i] = e < half * half ? e / half : -1;
    bb[i] = e - (ba[i] < 0 ? 0 : ba[i]) * half;
  }
  int cur = 0;
  for (int sweep = 0; sweep < 40 && k > 1; ++sweep) {
    double off = 0.0, dg = 0.0, sig = 0.0;
    for (int e = t; e < k * k; e += blockDim.x) {
      const int i = e / k, j = e % k;
      const double a = A[cur][i][j];
      if (i != j) off += a * a;
      else dg += a * a;
      if (i < j && jacobi_significant(a, A[cur][i][i], A[cur][j][j])) sig += 1.0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      off += __shfl_xor(off, o, 64);
      dg += __shfl_xor(dg, o, 64);
      sig += __shfl_xor(sig, o, 64);
    }
    double(*rd)[4] = red[sweep & 1];  // two copies: the next check writes the other one
    if ((t & 63) == 0) {
      rd[0][t >> 6] = off;
      rd[1][t >> 6] = dg;
      rd[2][t >> 6] = sig;
    }
    __syncthreads();
    const double offsum = (rd[0][0] + rd[0][1]) + (rd[0][2] + rd[0][3]);
    const double dgsum = (rd[1][0] + rd[1][1]) + (rd[1][2] + rd[1][3]);
    const double nsig = (rd[2][0] + rd[2][1]) + (rd[2][2] + rd[2][3]);
    if (nsig == 0.0 || offsum <= 1e-32 * (dgsum > 1e-300 ? dgsum : 1e-300)) break;  // uniform
    for (int round = 0; round < n - 1; ++round) {
      const double(*Ai)[65] = A[cur];
      const double(*Vi)[65] = V[cur];
      double(*Ao)[65] = A[cur ^ 1];
      double(*Vo)[65] = V[cur ^ 1];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (ba[i] < 0) continue;
        int pa, qa, pb, qb;
        jacobi_pair(round, ba[i], n, pa, qa);
        jacobi_pair(round, bb[i], n, pb, qb);
        const bool va = qa < k, vb = qb < k;  // false: the pair holds the padding index
        double ca = 1.0, sa = 0.0, cb = 1.0, sb = 0.0;
        if (va) jacobi_angle(Ai, pa, qa, ca, sa);
        if (vb) jacobi_angle(Ai, pb, qb, cb, sb);
        double x00 = Ai[pa][pb], x01 = vb ? Ai[pa][qb] : 0.0;
        double x10 = va ? Ai[qa][pb] : 0.0, x11 = (va && vb) ? Ai[qa][qb] : 0.0;
        double w00 = Vi[pa][pb], w01 = vb ? Vi[pa][qb] : 0.0;
        double w10 = va ? Vi[qa][pb] : 0.0, w11 = (va && vb) ? Vi[qa][qb] : 0.0;
        if (va) {  // rows p_a, q_a
          const double y00 = ca * x00 - sa * x10, y10 = sa * x00 + ca * x10;
          const double y01 = ca * x01 - sa * x11, y11 = sa * x01 + ca * x11;
          x00 = y00;
          x10 = y10;
          x01 = y01;
          x11 = y11;
        }
        if (vb) {  // columns p_b, q_b of A and of V
          const double y00 = cb * x00 - sb * x01, y01 = sb * x00 + cb * x01;
          const double y10 = cb * x10 - sb * x11, y11 = sb * x10 + cb * x11;
          x00 = y00;
          x01 = y01;
          x10 = y10;
          x11 = y11;
          const double z00 = cb * w00 - sb * w01, z01 = sb * w00 + cb * w01;
          const double z10 = cb * w10 - sb * w11, z11 = sb * w10 + cb * w11;
          w00 = z00;
          w01 = z01;
          w10 = z10;
          w11 = z11;
        }
        Ao[pa][pb] = x00;
        Vo[pa][pb] = w00;
        if (vb) {
          Ao[pa][qb] = x01;
          Vo[pa][qb] = w01;
        }
        if (va) {
          Ao[qa][pb] = x10;
          Vo[qa][pb] = w10;
        }
        if (va && vb) {
          Ao[qa][qb] = x11;
          Vo[qa][qb] = w11;
        }
      }
      __syncthreads();
      cur ^= 1;
    }
  }
  // ascending order of the eigenvalues, equal ones by index (a NaN counts as
  // +inf, so the ranks are a permutation): each thread ranks one value against
  // all k (independent LDS reads instead of a serial sort on one thread)
  for (int j = t; j < k; j += blockDim.x) {
    const double dj = A[cur][j][j], kj = dj == dj ? dj : INFINITY;
    int rank = 0;
    for (int i = 0; i < k; ++i) {
      const double di = A[cur][i][i], ki = di == di ? di : INFINITY;
      rank += (ki < kj || (ki == kj && i < j)) ? 1 : 0;
    }
    order[rank] = j;
  }
  __syncthreads();
  for (int e = t; e < k * k; e += blockDim.x) {
    int j = e / k, i = e % k;  // eigenvector j, component i
    evecs[(long)j * k + i] = V[cur][i][order[j]];
  }
  for (int j = t; j < k; j += blockDim.x) evals[j] = A[cur][order[j]][order[j]];
}

// Subspace rotation in place: V[:, i] = sum_j V[:, j] Y[i * k + j] for i < keep
// (columns of V are vectors of length n, stride ldv; Y holds k-vectors one after
// another).  Rows are independent: each thread reads all k entries of its row
// before writing the keep new ones, so the update is safe in place.
constexpr int kRotMax = 16;
__global__ __launch_bounds__(256) void subspace_rotate_kernel(double* __restrict__ V, long ldv, int k,
                                                              const double* __restrict__ Y, int keep, long n) {
  __shared__ double Ys[64 * kRotMax];
  for (int e = threadIdx.x; e < 64 * kRotMax; e += blockDim.x) {
    const int j = e / kRotMax, i = e % kRotMax;
    Ys[e] = (j < k && i < keep) ? Y[(long)i * k + j] : 0.0;
  }
  __syncthreads();
  for (long r = (long)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (long)gridDim.x * blockDim.x) {
    double acc[kRotMax];
#pragma unroll
    for (int i = 0; i < kRotMax; ++i) acc[i] = 0.0;
    for (int j = 0; j < k; ++j) {
      const double v = V[(long)j * ldv + r];
#pragma unroll
      for (int i = 0; i < kRotMax; ++i) acc[i] += v * Ys[j * kRotMax + i];
    }
#pragma unroll
    for (int i = 0; i < kRotMax; ++i)
      if (i < keep) V[(long)i * ldv + r] = acc[i];
  }
}

__global__ void f64_to_f32_kernel(const double* x, float* y, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = (float)x[i];
}
__global__ void f64_to_bf16_kernel(const double* x, uint16_t* y, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = f2bf((float)x[i]);
}
__global__ void f32_to_f64_kernel(const float* x, double* y, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = (double)x[i];
}

__global__ void diag_kernel(double* __restrict__ out, const DiagBlock* __restrict__ blocks,
                            const DiagTerm* __restrict__ terms) {
  const DiagBlock b = blocks[blockIdx.x];
  for (int e = threadIdx.x; e < b.rows * b.cols; e += blockDim.x) {
    int i = e / b.cols, j = e % b.cols;
    double acc = 0.0;
    for (int tt = b.t0; tt < b.t1; ++tt) {
      const DiagTerm& d = terms[tt];
      acc += d.w * d.x[i] * d.y[j];
    }
    out[b.out_off + (long)i * b.ld + j] = acc;
  }
}

// desc: src_off, ld, n, dst_off
__global__ void extract_diag_kernel(const int64_t* __restrict__ desc, const double* __restrict__ src,
                                    double* __restrict__ dst) {
  const int64_t* d = desc + 4 * blockIdx.x;
  for (int i = threadIdx.x; i < (int)d[2]; i += blockDim.x) dst[d[3] + i] = src[d[0] + (long)i * (d[1] + 1)];
}

inline int grid_for(long n, int bs = 256, int cap = 4096) {
  long g = (n + bs - 1) / bs;
  if (g < 1) g = 1;
  return (int)(g > cap ? cap : g);
}

}  // namespace

void launch_gemm_w32(int mode, bool buf, const GemmUnit* units, int n_units, const GemmItem* items, hipStream_t s) {
  if (n_units <= 0) return;
  dim3 grid((n_units + 3) / 4), block(256);
  if (mode == GEMM_TN) gemm_f64_w32<GEMM_TN, false><<<grid, block, 0, s>>>(units, items, n_units);
  else if (mode == GEMM_NN && buf) gemm_f64_w32<GEMM_NN, true><<<grid, block, 0, s>>>(units, items, n_units);
  else if (mode == GEMM_NN) gemm_f64_w32<GEMM_NN, false><<<grid, block, 0, s>>>(units, items, n_units);
  else if (buf) gemm_f64_w32<GEMM_NT, true><<<grid, block, 0, s>>>(units, items, n_units);
  else gemm_f64_w32<GEMM_NT, false><<<grid, block, 0, s>>>(units, items, n_units);
}

void launch_grad_expand(const GradView& v, bool left, const double* env, const double* site, double* out,
                        GemmUnit* units, GemmItem* items, hipStream_t s) {
  if (v.units > 0)
    grad_expand_kernel<<<grid_for(v.units), 256, 0, s>>>(v, left ? 1 : 0, env, site, out, units, items);
}

// tiles are at most 64 x 64 = 16 chunks of 256 elements
constexpr int kReduceChunks = 16;

void launch_splitk_reduce(const SplitTile* tiles, int n, const double* slots, hipStream_t s) {
  if (n > 0) splitk_reduce<<<dim3(n, kReduceChunks), 256, 0, s>>>(tiles, slots);
}

void launch_splitk_reduce_f32(const SplitTile* tiles, int n, const float* slots, hipStream_t s) {
  if (n > 0) splitk_reduce_f32<<<dim3(n, kReduceChunks), 256, 0, s>>>(tiles, slots);
}

void launch_gemm(int prec, int mode, const GemmUnit* units, int n_units, const GemmItem* items,
                 hipStream_t s) {
  if (n_units <= 0) return;
  dim3 grid(n_units), block(256);
  if (prec == PREC_F64) {
    if (mode == GEMM_NN) gemm_f64<GEMM_NN><<<grid, block, 0, s>>>(units, items);
    else if (mode == GEMM_NT) gemm_f64<GEMM_NT><<<grid, block, 0, s>>>(units, items);
    else gemm_f64<GEMM_TN><<<grid, block, 0, s>>>(units, items);
  } else if (prec == PREC_F32) {
    if (mode == GEMM_NN) gemm_f32<GEMM_NN, float, float><<<grid, block, 0, s>>>(units, items);
    else if (mode == GEMM_NT) gemm_f32<GEMM_NT, float, float><<<grid, block, 0, s>>>(units, items);
    else gemm_f32<GEMM_TN, float, float><<<grid, block, 0, s>>>(units, items);
  } else {  // PREC_BF16; no TN
    if (mode == GEMM_NN) gemm_bf16<GEMM_NN><<<grid, block, 0, s>>>(units, items);
    else gemm_bf16<GEMM_NT><<<grid, block, 0, s>>>(units, items);
  }
}

void launch_premix(double* out, const double* const* srcs, const int* ptr, const double* coef,
                   int n_out, long nnz, hipStream_t s) {
  if (n_out <= 0 || nnz <= 0) return;
  dim3 grid(grid_for(nnz, 256, 64), n_out);
  premix_kernel<<<grid, 256, 0, s>>>(out, srcs, ptr, coef, nnz);
}

void launch_pairmix(double* out, const double* const* srcs, const int* ptr, const double* coef, const long* out_off,
                    const int* nnz, int n_groups, hipStream_t s) {
  if (n_groups > 0) pairmix_kernel<<<n_groups, 256, 0, s>>>(out, srcs, ptr, coef, out_off, nnz);
}

void launch_fill(double* x, long n, double v, hipStream_t s) {
  if (n <= 0) return;
  fill_kernel<<<grid_for(n), 256, 0, s>>>(x, n, v);
}

void launch_copy_blocks(const int64_t* desc, int n_blocks, const double* src, double* dst,
                        hipStream_t s) {
  if (n_blocks <= 0) return;
  copy_blocks_kernel<<<n_blocks, 256, 0, s>>>(desc, src, dst);
}

void launch_axpy_dev(double* y, const double* x, const double* a, double sign, long n, hipStream_t s) {
  if (n > 0) axpy_dev_kernel<<<grid_for(n), 256, 0, s>>>(y, x, a, sign, n);
}

void launch_copy(double* dst, const double* src, long n, hipStream_t s) {
  if (n > 0) copy_kernel<<<grid_for(n), 256, 0, s>>>(dst, src, n);
}

void launch_fill_f32(float* x, long n, hipStream_t s) {
  if (n > 0) fill_f32_kernel<<<grid_for(n), 256, 0, s>>>(x, n);
}

void launch_dots(const double* V, long ldv, int k, const double* x, long n, double* partial,
                 double* out, hipStream_t s) {
  if (k <= 0) return;
  if (n <= kDotsOne) {
    dots_one<<<k, 512, 0, s>>>(V, ldv, x, n, out);
    return;
  }
  long chunk = 8192;
  int nchunk = (int)((n + chunk - 1) / chunk);
  if (nchunk > 512) {
    nchunk = 512;
    chunk = (n + nchunk - 1) / nchunk;
  }
  if (nchunk < 1) nchunk = 1;
  dots_partial<<<dim3(nchunk, k), 256, 0, s>>>(V, ldv, x, n, chunk, partial);
  dots_final<<<k, 256, 0, s>>>(partial, nchunk, out);
}

void launch_gemv(const double* V, long ldv, int k, const double* coef, double alpha, double* out,
                 double beta, long n, hipStream_t s) {
  gemv_kernel<<<grid_for(n), 256, 0, s>>>(V, ldv, k, coef, alpha, out, beta, n);
}

void launch_scale_by_norm(double* x, long n, const double* nrm2, hipStream_t s) {
  scale_by_norm_kernel<<<grid_for(n), 256, 0, s>>>(x, n, nrm2);
}

void launch_precond_diag(const double* r, const double* diag, const double* theta, double* out,
                         long n, hipStream_t s) {
  precond_diag_kernel<<<grid_for(n), 256, 0, s>>>(r, diag, theta, out, n);
}

void launch_shift_entries(const double* src, void* dst, bool bf16, const long* idx, const double* w, long n,
                          double shift, hipStream_t s) {
  if (n > 0) shift_entries_kernel<<<grid_for(n), 256, 0, s>>>(src, dst, bf16 ? 1 : 0, idx, w, n, shift);
}

void launch_axpy_ratio(double* y, const double* x, const double* num, const double* den, double sign, long n,
                       hipStream_t s) {
  if (n > 0) axpy_ratio_kernel<<<grid_for(n), 256, 0, s>>>(y, x, num, den, sign, n);
}

void launch_xpby_ratio(double* p, const double* z, const double* num, const double* den, long n, hipStream_t s) {
  if (n > 0) xpby_ratio_kernel<<<grid_for(n), 256, 0, s>>>(p, z, num, den, n);
}

void launch_axpy(double* y, const double* x, double a, long n, hipStream_t s) {
  if (n > 0) axpy_kernel<<<grid_for(n), 256, 0, s>>>(y, x, a, n);
}

void launch_add_squares(double* d, const double* V, long ldv, int k, long n, hipStream_t s) {
  if (n > 0 && k > 0) add_squares_kernel<<<grid_for(n), 256, 0, s>>>(d, V, ldv, k, n);
}

void launch_subspace_rotate(double* V, long ldv, int k, const double* Y, int keep, long n, hipStream_t s) {
  if (n <= 0 || keep <= 0) return;
  if (k > 64 || keep > kRotMax || keep > k) throw std::runtime_error("subspace rotation: k <= 64, keep <= 16 and <= k");
  subspace_rotate_kernel<<<grid_for(n), 256, 0, s>>>(V, ldv, k, Y, keep, n);
}

void launch_jacobi_eig(const double* G, int ldg, int k, double* evals, double* evecs,
                       hipStream_t s) {
  if (k > 64) throw std::runtime_error("subspace eigensolver: k <= 64");
  if (k > 0) jacobi_eig_kernel<<<1, 256, 0, s>>>(G, ldg, k, evals, evecs);
}

void launch_f64_to_f32(const double* x, float* y, long n, hipStream_t s) {
  if (n > 0) f64_to_f32_kernel<<<grid_for(n), 256, 0, s>>>(x, y, n);
}
void launch_f64_to_bf16(const double* x, uint16_t* y, long n, hipStream_t s) {
  if (n > 0) f64_to_bf16_kernel<<<grid_for(n), 256, 0, s>>>(x, y, n);
}
void launch_f32_to_f64(const float* x, double* y, long n, hipStream_t s) {
  if (n > 0) f32_to_f64_kernel<<<grid_for(n), 256, 0, s>>>(x, y, n);
}

void launch_diag(double* out, const DiagBlock* blocks, int n_blocks, const DiagTerm* terms,
                 hipStream_t s) {
  if (n_blocks > 0) diag_kernel<<<n_blocks, 256, 0, s>>>(out, blocks, terms);
}

void launch_extract_diag(const int64_t* desc, int n, const double* src, double* dst,
                         hipStream_t s) {
  if (n > 0) extract_diag_kernel<<<n, 64, 0, s>>>(desc, src, dst);
}

}  // namespace dmrg
