// Learned Davidson preconditioner on gfx950: network kernels (forward, cosine
// loss, backward, Adam), per-amplitude feature kernels and the gathering of
// training triples.  Element-wise kernels and deterministic column reductions
// (fixed chunks, partials summed in order); the hidden layer's products run on
// mlp_gemm_kernel, those of few rows and of bf16 widths other than 256 on the
// plain 64 x 64 tiles of kernels.hip (see mlp_net.cpp).
#include <hip/hip_runtime.h>

#include <algorithm>

#include <cmath>
#include <cstring>

#include "mlp.hpp"

namespace dmrg {

namespace {

constexpr int kThreads = 256;

inline int grid_of(long n) {
  long g = (n + kThreads - 1) / kThreads;
  return (int)(g < 1 ? 1 : (g > 65536 ? 65536 : g));
}

__device__ inline uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline double wave_min(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}

// Sum (or min) over the 256 threads of a block, same order on every call.
__device__ inline double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double r = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return r;
}
__device__ inline double block_min(double v, double* sh) {
  v = wave_min(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double r = fmin(fmin(sh[0], sh[1]), fmin(sh[2], sh[3]));
  __syncthreads();
  return r;
}

__global__ void layer1_kernel(const float* __restrict__ X, long n, int nin, const float* __restrict__ W1,
                              const float* __restrict__ b1, int width, float* __restrict__ a1,
                              uint16_t* __restrict__ a1b) {
  const long total = n * width;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (long)gridDim.x * blockDim.x) {
    const long i = e / width;
    const int j = (int)(e - i * width);
    float z = b1[j];
    for (int f = 0; f < nin; ++f) z = fmaf(X[i * nin + f], W1[j * nin + f], z);
    z = fmaxf(z, 0.f);
    if (a1) a1[e] = z;
    if (a1b) a1b[e] = bf16_rne(z);
  }
}

// One wave per row.
__global__ void layer3_kernel(float* __restrict__ z2, long n, int width, const float* __restrict__ b2,
                              const float* __restrict__ W3, const float* __restrict__ b3, float* __restrict__ y,
                              int store) {
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= n) return;
  float* zr = z2 + row * width;
  double acc = 0.0;
  for (int j = lane; j < width; j += 64) {
    float a = fmaxf(zr[j] + b2[j], 0.f);
    acc += (double)a * W3[j];
    if (store) zr[j] = a;
  }
  acc = wave_sum(acc);
  if (lane == 0) y[row] = (float)(acc + b3[0]);
}

// Fused bf16 inference of the width-256 network, y = W3 relu(W2 relu(W1 x + b1)
// + b2) + b3, without writing activations to memory.  Persistent workgroups of
// 8 waves (one per CU: W2 in bf16, 256 x 256, is staged once in LDS with a row
// pitch of 260) walk 32-row tiles: the tile's inputs are staged in LDS; layer 1
// (thread t: columns 4 (t % 64).. whose W1 rows it keeps in registers, rows
// 4 (t / 64)..) writes bf16 to LDS, the rounding the layered path applies;
// layer 2 runs on v_mfma_f32_16x16x16 bf16 (wave w: rows 16 (w & 1).., columns
// 64 (w >> 1)..: 4 tiles of 16 x 16); layer 3 is a dot product with W3 reduced
// over lanes and the four column quarters.
constexpr int kInfW = 256, kInfRows = 32, kInfPitch = kInfW + 4, kInfThreads = 512, kInfMaxIn = 16;
typedef short v4s_t __attribute__((ext_vector_type(4)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(kInfThreads) void mlp_infer_bf16_kernel(
    const float* __restrict__ X, long n, int nin, const float* __restrict__ W1, const float* __restrict__ b1,
    const uint16_t* __restrict__ W2b, const float* __restrict__ b2, const float* __restrict__ W3,
    const float* __restrict__ b3, float* __restrict__ y) {
  __shared__ __align__(16) uint16_t W2s[kInfW * kInfPitch];
  __shared__ __align__(16) uint16_t A1s[kInfRows * kInfPitch];
  __shared__ float Xs[kInfRows * kInfMaxIn];
  __shared__ float part[4][kInfRows];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int e = tid; e < kInfW * kInfW / 4; e += kInfThreads) {  // 4 bf16 (8 bytes) per step
    const int j = e / (kInfW / 4), i4 = (e % (kInfW / 4)) * 4;
    *reinterpret_cast<uint2*>(W2s + j * kInfPitch + i4) = *reinterpret_cast<const uint2*>(W2b + (long)j * kInfW + i4);
  }
  // layer-1 role of this thread: columns c0..c0+3, rows r0..r0+3 of every tile
  const int c0 = 4 * (tid & 63), r0 = 4 * (tid >> 6);
  float w1[4][kInfMaxIn], bb[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    bb[c] = b1[c0 + c];
#pragma unroll
    for (int f = 0; f < kInfMaxIn; ++f) w1[c][f] = f < nin ? W1[(c0 + c) * nin + f] : 0.f;
  }
  const int rb = wave & 1, cb = (wave >> 1) * 64;
  const long ntiles = (n + kInfRows - 1) / kInfRows;
  for (long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const long row0 = tile * kInfRows;
    __syncthreads();  // W2s staged / the previous tile's Xs, A1s and part[] read
    for (int e = tid; e < kInfRows * kInfMaxIn; e += kInfThreads) {
      const int r = e / kInfMaxIn, f = e % kInfMaxIn;
      Xs[e] = (f < nin && row0 + r < n) ? X[(row0 + r) * nin + f] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int r = r0 + rr;
      float z[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) z[c] = bb[c];
#pragma unroll
      for (int f = 0; f < kInfMaxIn; ++f) {
        const float xf = Xs[r * kInfMaxIn + f];
#pragma unroll
        for (int c = 0; c < 4; ++c) z[c] = fmaf(xf, w1[c][f], z[c]);
      }
      uint2 pk;
      pk.x = (uint32_t)bf16_rne(fmaxf(z[0], 0.f)) | ((uint32_t)bf16_rne(fmaxf(z[1], 0.f)) << 16);
      pk.y = (uint32_t)bf16_rne(fmaxf(z[2], 0.f)) | ((uint32_t)bf16_rne(fmaxf(z[3], 0.f)) << 16);
      *reinterpret_cast<uint2*>(A1s + r * kInfPitch + c0) = pk;
    }
    __syncthreads();
    v4f_t acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = (v4f_t){0.f, 0.f, 0.f, 0.f};
    const int ar = rb * 16 + (lane & 15);
#pragma unroll 4
    for (int k0 = 0; k0 < kInfW; k0 += 16) {
      const int kk = k0 + 4 * (lane >> 4);
      const uint2 av = *reinterpret_cast<const uint2*>(A1s + ar * kInfPitch + kk);
      v4s_t a;
      a[0] = (short)(av.x & 0xffff);
      a[1] = (short)(av.x >> 16);
      a[2] = (short)(av.y & 0xffff);
      a[3] = (short)(av.y >> 16);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int j = cb + 16 * t + (lane & 15);  // B[k][col j] = W2[j][k]
        const uint2 bv = *reinterpret_cast<const uint2*>(W2s + j * kInfPitch + kk);
        v4s_t b;
        b[0] = (short)(bv.x & 0xffff);
        b[1] = (short)(bv.x >> 16);
        b[2] = (short)(bv.y & 0xffff);
        b[3] = (short)(bv.y >> 16);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[t], 0, 0, 0);
      }
    }
    // layer 3: element q of acc[t] is row 4 (lane >> 4) + q, column cb + 16 t + (lane & 15)
    float sq[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int j = cb + 16 * t + (lane & 15);
      const float bj = b2[j], wj = W3[j];
#pragma unroll
      for (int q = 0; q < 4; ++q) sq[q] = fmaf(fmaxf(acc[t][q] + bj, 0.f), wj, sq[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int m = 1; m < 16; m <<= 1) sq[q] += __shfl_xor(sq[q], m);
    if ((lane & 15) == 0)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[wave >> 1][rb * 16 + 4 * (lane >> 4) + q] = sq[q];
    __syncthreads();
    if (tid < kInfRows && row0 + tid < n)
      y[row0 + tid] = ((part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid])) + b3[0];
  }
}

__global__ void seg_stats_kernel(const float* __restrict__ y, const float* __restrict__ t, int seglen,
                                 double* __restrict__ stats) {
  __shared__ double sh[4];
  const long base = (long)blockIdx.x * seglen;
  double yt = 0, yy = 0, tt = 0;
  for (int i = threadIdx.x; i < seglen; i += blockDim.x) {
    double a = y[base + i], b = t[base + i];
    yt += a * b;
    yy += a * a;
    tt += b * b;
  }
  yt = block_sum(yt, sh);
  yy = block_sum(yy, sh);
  tt = block_sum(tt, sh);
  if (threadIdx.x == 0) {
    stats[3 * blockIdx.x] = yt;
    stats[3 * blockIdx.x + 1] = yy;
    stats[3 * blockIdx.x + 2] = tt;
  }
}

__global__ void cos_grad_kernel(const float* __restrict__ y, const float* __restrict__ t,
                                const double* __restrict__ stats, int nseg, int seglen, float* __restrict__ dy) {
  const long total = (long)nseg * seglen;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (long)gridDim.x * blockDim.x) {
    const long sgi = e / seglen;
    const double yt = stats[3 * sgi], yy = stats[3 * sgi + 1], tt = stats[3 * sgi + 2];
    double g = 0.0;
    if (yy > 0.0 && tt > 0.0) {
      const double ny = sqrt(yy), nt = sqrt(tt), c = yt / (ny * nt);
      g = -(t[e] / (ny * nt) - c * y[e] / yy) / nseg;
    }
    dy[e] = (float)g;
  }
}

__global__ void adam_kernel(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                            const float* __restrict__ g, long n, float lr, float b1, float b2, float eps, float c1,
                            float c2) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1, vh = vi / c2;
    w[i] -= lr * mh / (sqrtf(vh) + eps);
  }
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = bf16_rne(x[i]);
}

// Layer 1 for widths whose 4-column groups divide a workgroup: a thread keeps its
// four columns' weights in registers and walks rows (one 16-byte store per row);
// 64 MB of activations in 47 us instead of 246 (65536 rows, width 256).
constexpr int kL1MaxIn = 16;
__global__ __launch_bounds__(kThreads) void layer1_cols_kernel(const float* __restrict__ X, long n, int nin,
                                                               const float* __restrict__ W1,
                                                               const float* __restrict__ b1, int width,
                                                               float* __restrict__ a1) {
  const int ng = width >> 2, c0 = 4 * (threadIdx.x % ng);
  float w[4][kL1MaxIn], b[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    b[c] = b1[c0 + c];
#pragma unroll
    for (int f = 0; f < kL1MaxIn; ++f) w[c][f] = f < nin ? W1[(c0 + c) * nin + f] : 0.f;
  }
  const int nr = kThreads / ng;  // rows of a workgroup at a time
  constexpr int RU = 4;          // rows of a thread in flight
  for (long i0 = (long)blockIdx.x * nr * RU + threadIdx.x / ng; i0 < n; i0 += (long)gridDim.x * nr * RU) {
    float z[RU][4];
#pragma unroll
    for (int u = 0; u < RU; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) z[u][c] = b[c];
#pragma unroll
    for (int f = 0; f < kL1MaxIn; ++f)
      if (f < nin) {
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const long i = i0 + u * nr;
          const float x = X[(i < n ? i : n - 1) * nin + f];
#pragma unroll
          for (int c = 0; c < 4; ++c) z[u][c] = fmaf(x, w[c][f], z[u][c]);
        }
      }
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      const long i = i0 + u * nr;
      if (i < n) {
        float4 o = {fmaxf(z[u][0], 0.f), fmaxf(z[u][1], 0.f), fmaxf(z[u][2], 0.f), fmaxf(z[u][3], 0.f)};
        *reinterpret_cast<float4*>(a1 + i * width + c0) = o;
      }
    }
  }
}

// The hidden layer's products of a training step on v_mfma_f32_16x16x4f32, with
// the elementwise work around them fused in:
//  FWD: a2 = relu(a1 W2^T + b2), stored, and the layer-3 dot products of its rows
//       (fp64, one part per 64-column wave);
//  DA:  dz1 = (dz2 W2) (a1 > 0), never stored: its column sums with every input
//       feature and alone (dW1, db1) per 128-row tile;
//  DW:  dW2 = dz2^T a1 per chunk of kRowsDW rows, and in the first column tile the
//       column sums of dz2 (db2) and of dy a2 (dW3);
// dz2 = (a2 > 0) dy W3 is formed as it is loaded.  One 256-thread workgroup per
// 128 x TN tile, 16-deep slices through LDS, the next slice's loads in flight;
// each wave owns 64 x 64 (TN = 128) or 32 x 64 (TN = 64).  Operands stay in LDS
// as they come, [row][k] or [k][row], in row pitches without bank conflicts.
// MFMA step h takes k = 4 h .. 4 h + 3, so the pre-activations have the bits of
// any kernel that adds k in order, and the ReLU masks do not depend on the tile.
// Sums over rows run in fp64.  65536 rows of width 256: one training step 3.07 -> 0.53 ms
// (FWD 124 us, 69 TFLOP/s; DA 157 us; DW 99 us), the same bits; the 12 column-sum passes alone
// took 1.6 ms (128 workgroups, one row at a time).
enum MlpKind { MLP_FWD = 0, MLP_DA = 1, MLP_DW = 2 };
constexpr int kMT = 128, kMK = 16, kMPk = kMK + 4, kMPr = kMT + 4;
constexpr int kRowsDW = 512;
struct MlpArgs {
  const float *a1, *a2, *dy, *W2, *W3, *b2, *X;
  float *out;       // FWD: a2 (may be null), DW: chunk partials of dW2
  double *part;     // FWD: layer-3 parts [column wave][n]; DA: [row tile][width][nin + 1]; DW: [chunk][width][2]
  long n;
  int width, nin, vec, vecw;  // vec (vecw): activations (W2, W3) have 16-byte aligned rows
};

__device__ inline float4 row4(const float* __restrict__ p, int c, int width, int vec) {
  if (vec && c + 3 < width) return *reinterpret_cast<const float4*>(p + c);
  float4 v;
  v.x = c < width ? p[c] : 0.f;
  v.y = c + 1 < width ? p[c + 1] : 0.f;
  v.z = c + 2 < width ? p[c + 2] : 0.f;
  v.w = c + 3 < width ? p[c + 3] : 0.f;
  return v;
}

template <int KIND, int TN>
__global__ __launch_bounds__(256) void mlp_gemm_kernel(MlpArgs P) {
  constexpr int WC = TN / 64, WR = 4 / WC, RB = kMT / WR / 16;  // wave grid, row blocks of a wave
  constexpr int NAL = kMT * kMK / 4 / 256, NBL = TN * kMK / 4 / 256;
  __shared__ __align__(16) float As[kMT * kMPk];
  __shared__ __align__(16) float Bs[TN * kMPk];
  __shared__ double red[kMT][2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int wr = (wave / WC) * 16 * RB, wc = (wave % WC) * 64;
  const int W = P.width;
  const int n0 = blockIdx.y * TN;                                         // first column
  const long m0 = KIND == MLP_DW ? (long)blockIdx.z * kMT : (long)blockIdx.x * kMT;  // first row
  const long k0 = KIND == MLP_DW ? (long)blockIdx.x * kRowsDW : 0;
  const long K = KIND == MLP_DW ? (P.n - k0 < kRowsDW ? P.n - k0 : kRowsDW) : W;
  v4f_t acc[RB][4];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = (v4f_t){0.f, 0.f, 0.f, 0.f};
  double s2[4] = {0, 0, 0, 0}, s3[4] = {0, 0, 0, 0};  // DW: this thread's 4 columns of db2, dW3
  float4 ra[NAL], rb[NBL];
  const float4 zero = {0.f, 0.f, 0.f, 0.f};
  auto load = [&](long ks) {
#pragma unroll
    for (int j = 0; j < NAL; ++j) {
      const int e = tid + 256 * j;
      if constexpr (KIND == MLP_DW) {  // [k][row]: row k of a2, 4 columns (dz2's, this tile's rows of dW2)
        const int k = e / (kMT / 4), c = (int)m0 + 4 * (e % (kMT / 4));
        float4 v = zero;
        if (ks + k < K) {
          const long i = k0 + ks + k;
          const float4 a = row4(P.a2 + i * W, c, W, P.vec), w3 = row4(P.W3, c, W, P.vecw);
          const float d = P.dy[i];
          v.x = a.x > 0.f ? d * w3.x : 0.f;
          v.y = a.y > 0.f ? d * w3.y : 0.f;
          v.z = a.z > 0.f ? d * w3.z : 0.f;
          v.w = a.w > 0.f ? d * w3.w : 0.f;
          if (blockIdx.y == 0) {
            s2[0] += v.x;
            s2[1] += v.y;
            s2[2] += v.z;
            s2[3] += v.w;
            s3[0] += (double)a.x * d;
            s3[1] += (double)a.y * d;
            s3[2] += (double)a.z * d;
            s3[3] += (double)a.w * d;
          }
        }
        ra[j] = v;
      } else {  // [row][k]
        const int m = e / (kMK / 4), k = (int)ks + 4 * (e % (kMK / 4));
        float4 v = zero;
        if (m0 + m < P.n) {
          const long i = m0 + m;
          v = row4((KIND == MLP_FWD ? P.a1 : P.a2) + i * W, k, W, P.vec);
          if constexpr (KIND == MLP_DA) {
            const float d = P.dy[i];
            const float4 w3 = row4(P.W3, k, W, P.vecw);
            v.x = v.x > 0.f ? d * w3.x : 0.f;
            v.y = v.y > 0.f ? d * w3.y : 0.f;
            v.z = v.z > 0.f ? d * w3.z : 0.f;
            v.w = v.w > 0.f ? d * w3.w : 0.f;
          }
        }
        ra[j] = v;
      }
    }
#pragma unroll
    for (int j = 0; j < NBL; ++j) {
      const int e = tid + 256 * j;
      if constexpr (KIND == MLP_FWD) {  // W2[n][k]
        const int m = e / (kMK / 4), k = (int)ks + 4 * (e % (kMK / 4));
        rb[j] = n0 + m < W ? row4(P.W2 + (long)(n0 + m) * W, k, W, P.vecw) : zero;
      } else {  // [k][n]: W2 or a1
        const int k = e / (TN / 4), c = n0 + 4 * (e % (TN / 4));
        rb[j] = ks + k < K ? row4((KIND == MLP_DA ? P.W2 + (ks + k) * W : P.a1 + (k0 + ks + k) * W), c, W,
                                  KIND == MLP_DA ? P.vecw : P.vec)
                           : zero;
      }
    }
  };
  load(0);
  for (long ks = 0; ks < K; ks += kMK) {
    __syncthreads();  // the previous slice is read
#pragma unroll
    for (int j = 0; j < NAL; ++j) {
      const int e = tid + 256 * j;
      if constexpr (KIND == MLP_DW)
        *reinterpret_cast<float4*>(As + (e / (kMT / 4)) * kMPr + 4 * (e % (kMT / 4))) = ra[j];
      else
        *reinterpret_cast<float4*>(As + (e / (kMK / 4)) * kMPk + 4 * (e % (kMK / 4))) = ra[j];
    }
#pragma unroll
    for (int j = 0; j < NBL; ++j) {
      const int e = tid + 256 * j;
      if constexpr (KIND == MLP_FWD)
        *reinterpret_cast<float4*>(Bs + (e / (kMK / 4)) * kMPk + 4 * (e % (kMK / 4))) = rb[j];
      else
        *reinterpret_cast<float4*>(Bs + (e / (TN / 4)) * (TN + 4) + 4 * (e % (TN / 4))) = rb[j];
    }
    __syncthreads();
    if (ks + kMK < K) load(ks + kMK);
    float a[RB][4], b[4][4];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      if constexpr (KIND == MLP_DW) {
#pragma unroll
        for (int h = 0; h < 4; ++h) a[i][h] = As[(4 * h + kq) * kMPr + wr + 16 * i + r];
      } else {
#pragma unroll
        for (int h = 0; h < 4; ++h) a[i][h] = As[(wr + 16 * i + r) * kMPk + 4 * h + kq];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (KIND == MLP_FWD) {
#pragma unroll
        for (int h = 0; h < 4; ++h) b[j][h] = Bs[(wc + 16 * j + r) * kMPk + 4 * h + kq];
      } else {
#pragma unroll
        for (int h = 0; h < 4; ++h) b[j][h] = Bs[(4 * h + kq) * (TN + 4) + wc + 16 * j + r];
      }
    }
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][h], b[j][h], acc[i][j], 0, 0, 0);
  }
  // accumulator element q: row 4 kq + q of block i, column r of block j
  if constexpr (KIND == MLP_FWD) {
    float bj[4], wj[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = n0 + wc + 16 * j + r;
      bj[j] = c < W ? P.b2[c] : 0.f;
      wj[j] = c < W ? P.W3[c] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const long m = m0 + wr + 16 * i + 4 * kq + q;
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = n0 + wc + 16 * j + r;
          const float v = fmaxf(acc[i][j][q] + bj[j], 0.f);
          if (c < W) {
            s += (double)v * wj[j];
            if (P.out && m < P.n) P.out[m * W + c] = v;
          }
        }
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, 64);
        if (r == 0 && m < P.n) P.part[((long)blockIdx.y * WC + wave % WC) * P.n + m] = s;
      }
  } else if constexpr (KIND == MLP_DA) {
    // dz1 = da1 (a1 > 0), in place
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const long m = m0 + wr + 16 * i + 4 * kq + q;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = n0 + wc + 16 * j + r;
          if (!(m < P.n && c < W && P.a1[m * W + c] > 0.f)) acc[i][j][q] = 0.f;
        }
      }
    // column sums with every feature (the last one is 1), 16 features at a time:
    // the tile's inputs in LDS, the rows of a lane in order, then the 4 lane
    // groups, then the waves of the column strip
    const int nf = P.nin + 1;
    double* sh = &red[0][0];  // [WR][TN]
    for (int f0 = 0; f0 < nf; f0 += 16) {
      __syncthreads();  // As and red are read
      for (int e = tid; e < kMT * 16; e += 256) {
        const int m = e >> 4, f = f0 + (e & 15);
        As[(e & 15) * kMPr + m] = f < P.nin ? (m0 + m < P.n ? P.X[(m0 + m) * P.nin + f] : 0.f) : 1.f;
      }
      __syncthreads();
      for (int f = f0; f < nf && f < f0 + 16; ++f) {
        double s[4] = {0, 0, 0, 0};
        const float* xf = As + (f - f0) * kMPr + wr + 4 * kq;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          const float4 xv = *reinterpret_cast<const float4*>(xf + 16 * i);
          const double x[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) s[j] = fma((double)acc[i][j][q], x[q], s[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          s[j] += __shfl_xor(s[j], 16, 64);
          s[j] += __shfl_xor(s[j], 32, 64);
        }
        if (f > f0) __syncthreads();
        if (kq == 0)
#pragma unroll
          for (int j = 0; j < 4; ++j) sh[(wave / WC) * TN + wc + 16 * j + r] = s[j];
        __syncthreads();
        if (tid < TN && n0 + tid < W) {
          double t = 0.0;
          for (int w = 0; w < WR; ++w) t += sh[w * TN + tid];
          P.part[((long)blockIdx.x * W + n0 + tid) * nf + f] = t;
        }
      }
    }
  } else {
    float* out = P.out + (long)blockIdx.x * W * W;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const long m = m0 + wr + 16 * i + 4 * kq + q;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = n0 + wc + 16 * j + r;
          if (m < W && c < W) out[m * W + c] = acc[i][j][q];
        }
      }
    if (blockIdx.y == 0) {  // column group tid % 32, row groups tid / 32 added in order
      for (int g = 0; g < 8; ++g) {
        __syncthreads();
        if (tid / 32 == g)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            double* d = red[4 * (tid % 32) + c];
            d[0] = (g ? d[0] : 0.0) + s2[c];
            d[1] = (g ? d[1] : 0.0) + s3[c];
          }
      }
      __syncthreads();
      if (tid < kMT && m0 + tid < W) {
        double* d = P.part + ((long)blockIdx.x * W + m0 + tid) * 2;
        d[0] = red[tid][0];
        d[1] = red[tid][1];
      }
    }
  }
}

// y[i] = sum of its layer-3 parts + b3
__global__ void layer3_parts_kernel(const double* __restrict__ part, int np, long n, const float* __restrict__ b3,
                                    float* __restrict__ y) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int p = 0; p < np; ++p) s += part[p * n + i];
    y[i] = (float)(s + b3[0]);
  }
}

// Sums over chunks of partial[c][j], j = col ns + f: to o0[col os0 + f] for
// f < n0, to o1[col] for f = n0; 8 interleaved groups of chunks, each in order,
// added in order.
template <typename T>
__global__ __launch_bounds__(256) void sum_chunks_kernel(const T* __restrict__ partial, int nchunks, long len, int ns,
                                                         int n0, float* __restrict__ o0, long os0,
                                                         float* __restrict__ o1) {
  __shared__ double sh[8][32];
  const long j = (long)blockIdx.x * 32 + (threadIdx.x & 31);
  const int g = threadIdx.x >> 5;
  double acc = 0.0;
  if (j < len) {
#pragma unroll 8
    for (int c = g; c < nchunks; c += 8) acc += partial[(long)c * len + j];
  }
  sh[g][threadIdx.x & 31] = acc;
  __syncthreads();
  if (g == 0 && j < len) {
    for (int x = 1; x < 8; ++x) acc += sh[x][threadIdx.x & 31];
    const long col = j / ns;
    const int f = (int)(j - col * ns);
    if (f < n0) o0[col * os0 + f] = (float)acc;
    else o1[col] = (float)acc;
  }
}

// partial[b] = sum of the b-th kRowsDW elements of x
__global__ __launch_bounds__(256) void sum_rows_kernel(const float* __restrict__ x, long n, double* __restrict__ partial) {
  __shared__ double sh[4];
  const long b = (long)blockIdx.x * kRowsDW, e = b + kRowsDW < n ? b + kRowsDW : n;
  double acc = 0.0;
  for (long i = b + threadIdx.x; i < e; i += 256) acc += x[i];
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// one block per feature block: s_b = mean |d - theta|, then mean and min of (d - theta)/s_b
__global__ void feat_stats_kernel(const double* __restrict__ d, const double* __restrict__ theta,
                                  const int64_t* __restrict__ blocks, double* __restrict__ stats) {
  __shared__ double sh[4];
  const int64_t* b = blocks + 4 * blockIdx.x;
  const long off = b[0], ld = b[1];
  const int rows = (int)b[2], cols = (int)b[3];
  const long size = (long)rows * cols;
  const double th = theta[0];
  double sa = 0.0;
  for (long e = threadIdx.x; e < size; e += blockDim.x) {
    const long i = e / cols, j = e - i * cols;
    sa += fabs(d[off + i * ld + j] - th);
  }
  sa = block_sum(sa, sh);
  double s = sa / (double)size;
  if (!(s > 1e-300)) s = 1e-300;
  double su = 0.0, mn = INFINITY;
  for (long e = threadIdx.x; e < size; e += blockDim.x) {
    const long i = e / cols, j = e - i * cols;
    const double u = (d[off + i * ld + j] - th) / s;
    su += u;
    mn = fmin(mn, u);
  }
  su = block_sum(su, sh);
  mn = block_min(mn, sh);
  if (threadIdx.x == 0) {
    stats[4 * blockIdx.x] = s;
    stats[4 * blockIdx.x + 1] = su / (double)size;
    stats[4 * blockIdx.x + 2] = mn;
    stats[4 * blockIdx.x + 3] = log((double)size) / 10.0;
  }
}

__global__ void feat_fill_kernel(const double* __restrict__ r, const double* __restrict__ d,
                                 const double* __restrict__ theta, const double* __restrict__ t,
                                 const int64_t* __restrict__ blocks, const double* __restrict__ stats,
                                 const double* __restrict__ nrr, const double* __restrict__ ntt, long n, float kpos,
                                 float* __restrict__ X) {
  const int64_t* b = blocks + 4 * blockIdx.x;
  const long off = b[0], ld = b[1];
  const int rows = (int)b[2], cols = (int)b[3];
  const long size = (long)rows * cols;
  const double th = theta[0];
  const double s = stats[4 * blockIdx.x], mu = stats[4 * blockIdx.x + 1], mn = stats[4 * blockIdx.x + 2],
               lsz = stats[4 * blockIdx.x + 3];
  const double sq = sqrt((double)n);
  const double fr = nrr[0] > 0.0 ? sq / sqrt(nrr[0]) : 0.0;
  const double ft = ntt[0] > 0.0 ? sq / sqrt(ntt[0]) : 0.0;
  for (long e = threadIdx.x; e < size; e += blockDim.x) {
    const long i = e / cols, j = e - i * cols;
    const long p = off + i * ld + j;
    const double ev = d[p] - th;
    double inv = ev == 0.0 ? 10.0 : s / ev;
    inv = fmin(fmax(inv, -10.0), 10.0);
    float* x = X + p * 8;
    x[0] = (float)(r[p] * fr);
    x[1] = (float)(ev / s);
    x[2] = (float)inv;
    x[3] = (float)(t[p] * ft);
    x[4] = (float)mu;
    x[5] = (float)mn;
    x[6] = (float)lsz;
    x[7] = kpos;
  }
}

__global__ void gather_rows_kernel(const float* __restrict__ X, int nf, const int64_t* __restrict__ idx, int m,
                                   float* __restrict__ out) {
  const long total = (long)m * nf;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (long)gridDim.x * blockDim.x) {
    const long j = e / nf;
    const int f = (int)(e - j * nf);
    out[e] = X[idx[j] * nf + f];
  }
}

__global__ void triple_target_kernel(const double* __restrict__ psi_i, const double* __restrict__ psi_star,
                                     const double* __restrict__ cdev, const int64_t* __restrict__ idx, int m,
                                     float* __restrict__ out) {
  const double c = cdev[0];
  const double sg = c >= 0.0 ? 1.0 : -1.0;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < m; j += gridDim.x * blockDim.x) {
    const long p = idx[j];
    out[j] = (float)(sg * psi_star[p] - fabs(c) * psi_i[p]);
  }
}

}  // namespace

void launch_mlp_layer1(const float* X, long n, int nin, const float* W1, const float* b1, int width, float* a1,
                       uint16_t* a1b, hipStream_t s) {
  if (n <= 0) return;
  // a thread's weights take longer to load than few rows to form: from 2^18 activations
  // on (width 256: 1 row 37 us per forward against 41, 1332 rows 48.3 against 47.7, 3000 rows
  // 57 against 50; width 128: 1332 rows 33 against 35, 6000 rows 44 against 38)
  if (a1 && !a1b && width % 4 == 0 && kThreads % (width / 4) == 0 && nin <= kL1MaxIn && n * width >= (1L << 18)) {
    const long rows = kThreads / (width / 4);
    layer1_cols_kernel<<<(int)std::min<long>((n + 4 * rows - 1) / (4 * rows), 2048), kThreads, 0, s>>>(X, n, nin, W1, b1, width, a1);
    return;
  }
  layer1_kernel<<<grid_of(n * width), kThreads, 0, s>>>(X, n, nin, W1, b1, width, a1, a1b);
}
void launch_mlp_layer3(float* z2, long n, int width, const float* b2, const float* W3, const float* b3, float* y,
                       bool store, hipStream_t s) {
  if (n > 0) layer3_kernel<<<(int)((n + 3) / 4), kThreads, 0, s>>>(z2, n, width, b2, W3, b3, y, store ? 1 : 0);
}
bool launch_mlp_infer_bf16(const float* X, long n, int nin, const float* W1, const float* b1, int width,
                           const uint16_t* W2b, const float* b2, const float* W3, const float* b3, float* y,
                           hipStream_t s) {
  if (width != kInfW || nin < 1 || nin > kInfMaxIn) return false;
  if (n <= 0) return true;
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const long ntiles = (n + kInfRows - 1) / kInfRows;
  const int grid = (int)std::min<long>(ntiles, std::max(cus, 1));
  mlp_infer_bf16_kernel<<<grid, kInfThreads, 0, s>>>(X, n, nin, W1, b1, W2b, b2, W3, b3, y);
  return true;
}
void launch_seg_stats(const float* y, const float* t, int nseg, int seglen, double* stats, hipStream_t s) {
  if (nseg > 0) seg_stats_kernel<<<nseg, kThreads, 0, s>>>(y, t, seglen, stats);
}
void launch_cos_grad(const float* y, const float* t, const double* stats, int nseg, int seglen, float* dy,
                     hipStream_t s) {
  long n = (long)nseg * seglen;
  if (n > 0) cos_grad_kernel<<<grid_of(n), kThreads, 0, s>>>(y, t, stats, nseg, seglen, dy);
}
// Few 128-row tiles leave most of the chip idle and the tile's chain of MFMAs and
// its row sums in the open: below 64 of them the plain 64 x 64 tiles and a wave per
// row are faster (width 256: 1 row 37 us per call against 43, 1332 rows 48 against 54,
// 3000 rows, 48 tiles, 50 against 55; 6000 rows, 94 tiles, 72 against 61; width 512: 1332
// rows, 44 tiles, 74 against 81, 3000 rows, 96 tiles, 108 against 85).
bool mlp_few_tiles(long n, int width) {
  const int tn = width <= 64 ? 64 : 128;
  return ((n + kMT - 1) / kMT) * ((width + tn - 1) / tn) < 64;
}
int mlp_layer3_parts(int width) { return width <= 64 ? 1 : (width + 127) / 128 * 2; }
int mlp_row_tiles(long n) { return (int)((n + kMT - 1) / kMT); }
int mlp_row_chunks(long n) { return (int)((n + kRowsDW - 1) / kRowsDW); }
template <typename T>
static void launch_sum_chunks(const T* partial, int nchunks, long len, int ns, int n0, float* o0, long os0, float* o1,
                              hipStream_t s) {
  sum_chunks_kernel<T><<<(int)((len + 31) / 32), 256, 0, s>>>(partial, nchunks, len, ns, n0, o0, os0, o1);
}
void launch_sum_all(const float* x, long n, double* part, float* out, hipStream_t s) {
  if (n <= 0) return;
  const int nch = mlp_row_chunks(n);
  sum_rows_kernel<<<nch, 256, 0, s>>>(x, n, part);
  launch_sum_chunks(part, nch, 1, 1, 1, out, 1, nullptr, s);
}
template <int KIND>
static void launch_mlp_gemm(const MlpArgs& P, hipStream_t s) {
  const int W = P.width, mt = (int)((P.n + kMT - 1) / kMT), tn = W <= 64 ? 64 : 128, nt = (W + tn - 1) / tn;
  const int nch = (int)((P.n + kRowsDW - 1) / kRowsDW);
  const dim3 grid = KIND == MLP_DW ? dim3(nch, nt, (W + kMT - 1) / kMT) : dim3(mt, nt);
  if (tn == 64) mlp_gemm_kernel<KIND, 64><<<grid, 256, 0, s>>>(P);
  else mlp_gemm_kernel<KIND, 128><<<grid, 256, 0, s>>>(P);
}
void launch_mlp_forward_f32(const float* a1, long n, int width, const float* W2, const float* b2, const float* W3,
                            const float* b3, float* a2, double* part, float* y, hipStream_t s) {
  if (n <= 0) return;
  MlpArgs P{};
  P.a1 = a1, P.W2 = W2, P.W3 = W3, P.b2 = b2, P.out = a2, P.part = part, P.n = n, P.width = width;
  P.vec = width % 4 == 0;
  P.vecw = P.vec && ((uintptr_t)W2 | (uintptr_t)W3) % 16 == 0;
  launch_mlp_gemm<MLP_FWD>(P, s);
  layer3_parts_kernel<<<grid_of(n), kThreads, 0, s>>>(part, mlp_layer3_parts(width), n, b3, y);
}
void launch_mlp_backward_f32(const float* X, int nin, const float* a1, const float* a2, const float* dy, long n,
                             int width, const float* W2, const float* W3, double* part, float* gpart, float* gW1,
                             float* gb1, float* gW2, float* gb2, float* gW3, hipStream_t s) {
  if (n <= 0) return;
  MlpArgs P{};
  P.a1 = a1, P.a2 = a2, P.dy = dy, P.W2 = W2, P.W3 = W3, P.X = X, P.n = n, P.width = width, P.nin = nin;
  P.vec = width % 4 == 0;
  P.vecw = P.vec && ((uintptr_t)W2 | (uintptr_t)W3) % 16 == 0;
  const int nch = mlp_row_chunks(n), mt = mlp_row_tiles(n);
  P.out = gpart, P.part = part;
  launch_mlp_gemm<MLP_DW>(P, s);
  launch_sum_chunks(gpart, nch, (long)width * width, 1, 1, gW2, 1, nullptr, s);
  launch_sum_chunks(part, nch, 2L * width, 2, 1, gb2, 1, gW3, s);
  P.out = nullptr;  // the parts are reused: the sums above come first on the stream
  launch_mlp_gemm<MLP_DA>(P, s);
  launch_sum_chunks(part, mt, (long)(nin + 1) * width, nin + 1, nin, gW1, nin, gb1, s);
}
void launch_adam(float* w, float* m, float* v, const float* g, long n, float lr, float b1, float b2, float eps,
                 float c1, float c2, hipStream_t s) {
  if (n > 0) adam_kernel<<<grid_of(n), kThreads, 0, s>>>(w, m, v, g, n, lr, b1, b2, eps, c1, c2);
}
void launch_f32_to_bf16_rne(const float* x, uint16_t* y, long n, hipStream_t s) {
  if (n > 0) f32_to_bf16_kernel<<<grid_of(n), kThreads, 0, s>>>(x, y, n);
}
void launch_feat_stats(const double* d, const double* theta, const int64_t* blocks, int nb, double* stats,
                       hipStream_t s) {
  if (nb > 0) feat_stats_kernel<<<nb, kThreads, 0, s>>>(d, theta, blocks, stats);
}
void launch_feat_fill(const double* r, const double* d, const double* theta, const double* t,
                      const int64_t* blocks, int nb, const double* stats, const double* nrr, const double* ntt,
                      long n, float kpos, float* X, hipStream_t s) {
  if (nb > 0) feat_fill_kernel<<<nb, kThreads, 0, s>>>(r, d, theta, t, blocks, stats, nrr, ntt, n, kpos, X);
}
void launch_gather_rows(const float* X, int nf, const int64_t* idx, int m, float* out, hipStream_t s) {
  if (m > 0) gather_rows_kernel<<<grid_of((long)m * nf), kThreads, 0, s>>>(X, nf, idx, m, out);
}
void launch_triple_target(const double* psi_i, const double* psi_star, const double* cdev, const int64_t* idx,
                          int m, float* out, hipStream_t s) {
  if (m > 0) triple_target_kernel<<<grid_of(m), kThreads, 0, s>>>(psi_i, psi_star, cdev, idx, m, out);
}

}  // namespace dmrg
