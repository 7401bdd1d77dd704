// Device kernels (gfx950) and their host launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace dmrg {

// One product term of a grouped block GEMM: acc += coef * op(A) * op(B), K deep.
struct GemmItem {
  const void* A;
  const void* B;
  int lda, ldb, K, pad;
  double coef;
};

// One output tile (rows m0.., cols n0.., at most 64 x 64) of an M x N output
// block; it accumulates items [ib, ie) in order (no atomics: deterministic).
// shape (one-wave and stream kernels): 8 RB + CB for a (16 RB) x (16 CB) tile, RB in
// 1..4, CB in 1..2 (one-wave kernel, 0 = 32 x 32) or 1..4 (stream kernel).
struct GemmUnit {
  void* C;
  int ldc, M, N, m0, n0, ib, ie, accumulate;
  int shape;
};

// Depth of item i of a unit's list [ib, ie), the last one's past its end, for kernels
// that look ahead.  0, and no read, where the list is empty: ib = ie may be 0, and
// items[-1] lies in front of the table.
__host__ __device__ inline int list_depth(const GemmItem* items, int i, int ib, int ie) {
  if (ib >= ie) return 0;
  return items[i < ie ? i : ie - 1].K;
}

enum GemmMode : int {
  GEMM_NN = 0,  // A: M x K row-major, B: K x N row-major
  GEMM_NT = 1,  // A: M x K row-major, B: N x K row-major (B transposed)
  GEMM_TN = 2,  // A: K x M row-major (A transposed), B: K x N row-major
};

// Element precision of A and B (C is fp64 for FP64, fp32 otherwise).
enum GemmPrec : int { PREC_F64 = 0, PREC_F32 = 1, PREC_BF16 = 2, PREC_BF16_A32 = 3 };

void launch_gemm(int prec, int mode, const GemmUnit* units, int n_units, const GemmItem* items,
                 hipStream_t s);

// fp64 one-wave variant (one wave per unit, tile of 16..64 rows by 16 or 32
// columns from the unit's shape, operands from global memory).  Units with accumulate == 2 write
// the full tile, row-major (tile rows x tile cols), to a partial slot (split-K).
// buf: NN / NT launch whose items all pass buffer_reach_ok (raw buffer loads);
// otherwise plain loads (and any mode).
void launch_gemm_w32(int mode, bool buf, const GemmUnit* units, int n_units, const GemmItem* items, hipStream_t s);
// Whether one item may take the buffer-load path: every element offset a tile
// forms from the operand starts (up to 32 past the last row's K, NN rows of B up
// to K + 32) stays below 1 GiB in bytes, so offsets fit 32-bit arithmetic.
inline bool buffer_reach_ok(int mode, int M, int N, int K, int lda, int ldb, size_t esz_a, size_t esz_b) {
  if (mode != GEMM_NN && mode != GEMM_NT) return false;
  const long lim = 1L << 30;
  const long ra = ((long)(M - 1) * lda + K + 32) * (long)esz_a;
  const long rb = (mode == GEMM_NT ? (long)(N - 1) * ldb + K + 32 : (long)(K + 32) * ldb + N) * (long)esz_b;
  return ra < lim && rb < lim;
}

// Row products of the integral gradient (grad.cpp), expanded into units and items
// on the device.  A job's rows (channels) all have the blocks blk0 .. blk0 + nblk
// and the tiles tile0 .. tile0 + ntile; row r's blocks start at out + r K of the
// output.  srcs[src0 + kind nblk + b]: block b's operands for the rows of a kind
// (env relative to the row's channel); unit u = u0 + r ntile + tile, item u (none
// where the block has no source: zeros are written).
struct GradJob {
  long u0, out, K;
  int ntile, tile0, blk0, nblk, src0, row0;
};
struct GradTile {
  int block, m0, n0, shape;
};
struct GradBlock {
  long off;
  int mi, mj;
};
struct GradSrc {
  long env, site;
  int K, lda, ldb, valid;
};
struct GradRow {
  long chan;
  int kind, pad;
};
struct GradView {
  const GradJob* jobs;
  const GradTile* tiles;
  const GradBlock* blocks;
  const GradSrc* srcs;
  const GradRow* rows;
  int n_jobs;
  long units;
};
// left: A = env block, B = site block; right: A = site block, B = env block.
void launch_grad_expand(const GradView& v, bool left, const double* env, const double* site, double* out,
                        GemmUnit* units, GemmItem* items, hipStream_t s);

// Output tile (rows m0.., cols n0.. of an M x N block, tm x tn <= 64 x 64
// elements) = sum of ns partial tiles (row-major tm x tn each) stored one after
// another from element s0 of the slot buffer, summed in order; acc = 1 adds
// that sum to the tile instead.
struct SplitTile {
  void* C;
  long s0;
  int ldc, M, N, m0, n0, ns, tm, tn;
  int acc, pad;
};
void launch_splitk_reduce(const SplitTile* tiles, int n, const double* slots, hipStream_t s);
// NT stream kernel (gemm_stream.hip; prec PREC_F64 or PREC_F32: operands,
// accumulation and outputs in that type; PREC_BF16_A32: A fp32, rounded to bf16 after
// the item's coefficient, B bf16, accumulation and outputs fp32): one wave per unit, tile (16 RB) x
// (16 CB) with RB = shape >> 3 and CB = shape & 7 in 1..4.  The operands lie in
// buffers with 64 readable bytes past their end (DevMem's slack); partial tiles
// (accumulate == 2) are 16 CB wide.
void launch_gemm_stream(int prec, int tag, const GemmUnit* units, int n_units, const GemmItem* items, hipStream_t s);
// Slab kernel (gemm_slab.hip): T_f = X_f B for the factors f of one block shape.  Job
// job0 + f: X_f (M x K, row-major, row stride K) and T_f (row stride ldt; fp64 for
// PREC_F64, fp32 otherwise).  A unit computes rows [row0, row1) of the factors' rows
// stacked (row f M + m) and columns n0 .. n0 + N (at most 64): boff is the
// element of B's row 0 and column n0 (row-major, row stride ldb).  X is read up to 15 bytes past its last element.
struct SlabJob {
  const void* X;
  void* T;
};
struct SlabUnit {
  long boff;
  int ldb, K, M, N, ldt, n0, job0, row0, row1;
};
// tall: waves of 32 rows (128 rows a step per workgroup), otherwise of 16.
void launch_gemm_slab(int prec, int tag, bool tall, const SlabUnit* units, int n_units, const SlabJob* jobs,
                      const void* B, hipStream_t s);
void launch_splitk_reduce_f32(const SplitTile* tiles, int n, const float* slots, hipStream_t s);
// out[f][j] = sum_{i in [ptr[f], ptr[f+1])} coef[i] * src[idx[i]][j], j < nnz.
void launch_premix(double* out, const double* const* srcs, const int* ptr, const double* coef,
                   int n_out, long nnz, hipStream_t s);

// Device ceilings: a register-only fp64 MFMA loop (out: n_blocks * 256 doubles;
// returns the flops launched) and a streaming copy of bytes (multiple of 16,
// 16-byte aligned buffers).
long launch_mfma_f64_peak(double* out, int n_blocks, int iters, hipStream_t s);
void launch_stream_copy(const void* src, void* dst, long bytes, hipStream_t s);
// Per group g: out[out_off[g] + j] = sum_{i in [ptr[g], ptr[g+1])} coef[i] * srcs[i][j], j < nnz[g].
void launch_pairmix(double* out, const double* const* srcs, const int* ptr, const double* coef, const long* out_off,
                    const int* nnz, int n_groups, hipStream_t s);
void launch_fill(double* x, long n, double v, hipStream_t s);
// desc per block (9 x int64): src_off, src_row_stride, src_col_stride, dst_off,
// dst_row_stride, dst_col_stride, rows, cols, scale (bits of a double)
void launch_copy_blocks(const int64_t* desc, int n_blocks, const double* src, double* dst,
                        hipStream_t s);
void launch_axpy_dev(double* y, const double* x, const double* a, double sign, long n, hipStream_t s);
void launch_copy(double* dst, const double* src, long n, hipStream_t s);

// Davidson helpers (all fp64, deterministic two-pass reductions).
void launch_dots(const double* V, long ldv, int k, const double* x, long n, double* partial,
                 double* out, hipStream_t s);
void launch_fill_f32(float* x, long n, hipStream_t s);
void launch_gemv(const double* V, long ldv, int k, const double* coef, double alpha,
                 double* out, double beta, long n, hipStream_t s);
void launch_scale_by_norm(double* x, long n, const double* nrm2, hipStream_t s);
void launch_precond_diag(const double* r, const double* diag, const double* theta, double* out,
                         long n, hipStream_t s);
// dst[idx[i]] = round(src[idx[i]] - w[i] * shift) into an fp32 (bf16 = false) or bf16 copy.
void launch_shift_entries(const double* src, void* dst, bool bf16, const long* idx, const double* w, long n,
                          double shift, hipStream_t s);
// y += a x
void launch_axpy(double* y, const double* x, double a, long n, hipStream_t s);
// y += sign * (num[0] / den[0]) x and p = z + (num[0] / den[0]) p (device scalars)
void launch_axpy_ratio(double* y, const double* x, const double* num, const double* den, double sign, long n,
                       hipStream_t s);
void launch_xpby_ratio(double* p, const double* z, const double* num, const double* den, long n, hipStream_t s);
// d[i] += sum_{j<k} V[j ldv + i]^2.
void launch_add_squares(double* d, const double* V, long ldv, int k, long n, hipStream_t s);
// In place: V[:, i] = sum_{j<k} V[:, j] Y[i k + j] for i < keep (k <= 64, keep <= 16).
void launch_subspace_rotate(double* V, long ldv, int k, const double* Y, int keep, long n, hipStream_t s);
void launch_jacobi_eig(const double* G, int ldg, int k, double* evals, double* evecs,
                       hipStream_t s);

// precision conversions
void launch_f64_to_f32(const double* x, float* y, long n, hipStream_t s);
void launch_f64_to_bf16(const double* x, uint16_t* y, long n, hipStream_t s);
void launch_f32_to_f64(const float* x, double* y, long n, hipStream_t s);

// H_eff diagonal: out[e] = sum_t w_t * xd[tx_t][ia] * yd[ty_t][ib] per block.
struct DiagBlock {
  long out_off;
  int ld, rows, cols, t0, t1;  // rows x cols block at out_off with row stride ld; terms [t0,t1)
};
struct DiagTerm {
  const double* x;  // diagonal of the left factor restricted to the block's row sector
  const double* y;  // diagonal of the right factor restricted to the block's col sector
  double w;
};
void launch_diag(double* out, const DiagBlock* blocks, int n_blocks, const DiagTerm* terms,
                 hipStream_t s);
// diag of each env block: out[j] = blk[j*(ld+1)], used to extract factor diagonals.
void launch_extract_diag(const int64_t* desc, int n, const double* src, double* dst,
                         hipStream_t s);

}  // namespace dmrg
