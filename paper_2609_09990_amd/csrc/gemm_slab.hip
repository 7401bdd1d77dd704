// Slab kernel: T_f = X_f psi for all factors f of one block shape (sigma phase A).
//
// Every left factor's block of one sector pair has the same shape (M x K) and
// multiplies the same slab of psi (K x N); only the matrices differ.  Taken block
// by block, CAS(20,20), M = 1024 had 713 thousand waves of mean K 42 that computed
// 770 elements each: 541 vector and 477 scalar instructions around 40 MFMAs.  Here
// the rows of all the factors are stacked: a unit is a range of stacked rows times a
// strip of at most 64 columns.
//
//  * The strip of psi goes through LDS 16 k's at a time, shared by the workgroup's
//    waves; a wave's row tile (16 RB rows) may span any number of factors, so that
//    rows are padded once per unit, not once per factor.
//  * Neighbouring lanes of a load or store take neighbouring bytes of a row: X goes
//    through the wave's own LDS in windows of 128 bytes a row, and T leaves as
//    column pairs, up to 256 bytes of a row from 16 lanes.  (X loaded in the MFMA
//    layout and T stored by rows, 16 bytes a lane: 64 L1 accesses per instruction,
//    2.7 times the write requests T needs, 2.5 ms.)  bf16 rows of X, 2-byte aligned,
//    are loaded in the MFMA layout.
//  * The next window is in flight while one is multiplied, across tiles; the next
//    tile's matrices are looked up a tile ahead.  Little LDS (31 KB) and few
//    registers, so that 16 or more waves share a CU: with the whole strip in LDS (64
//    k's) and eight waves of 32 rows, 1.74 ms; four waves of 64 rows, 1.93 ms.
//  * k order as in the one-wave kernels: fp64 / fp32 eight at a time (lane group
//    kq holds 2 kq and 2 kq + 1), at most four left over as one step; bf16 sixteen
//    at a time: fp32 and bf16 results keep their bits.
//
// Phase A at CAS(20,20), M = 1024: 2.8 -> 1.69 ms (random state; 2.87 -> 1.83 on that of
// a half sweep), of which writing the 4.5 GB of T takes 0.75 and the MFMAs 0.75; CAS(12,12), M = 512: 420 -> 272 us; CAS(16,16),
// M = 512, fp32: 388 -> 164 us, bf16: 376 -> 135 us.  (Storing a tile behind the next
// one's first loads, so that no load waits for stores, spills: 1.94 ms.)
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace dmrg {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef unsigned int v4ua __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int v3ua __attribute__((ext_vector_type(3), aligned(4)));
typedef unsigned int v2ua __attribute__((ext_vector_type(2), aligned(4)));

constexpr int KC = 16;  // k's of the strip in LDS, and of a window of X
constexpr int NW = 4;   // waves of a workgroup, 16 RB rows each

// KG: k's of one group; PITCH: row pitch of the strip, [k][column] (fp64, fp32: the
// lane groups of one read fall on different banks) or [column][k] (bf16).  VW: elements
// of X per lane and load (fp64, fp32: 16 bytes).
template <int P>
struct SlabElem;
template <>
struct SlabElem<PREC_F64> {
  typedef double in_t;
  typedef double out_t;
  typedef v4d acc_t;
  static constexpr int KG = 8, PITCH = 72, VW = 2;
  __device__ static int row(int kq, int q) { return kq + 4 * q; }  // accumulator element q of lane group kq
  __device__ static acc_t mfma(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
};
template <>
struct SlabElem<PREC_F32> {
  typedef float in_t;
  typedef float out_t;
  typedef v4f acc_t;
  static constexpr int KG = 8, PITCH = 80, VW = 4;
  __device__ static int row(int kq, int q) { return 4 * kq + q; }
  __device__ static acc_t mfma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};
template <>
struct SlabElem<PREC_BF16> {
  typedef uint16_t in_t;
  typedef float out_t;
  typedef v4f acc_t;
  static constexpr int KG = 16, PITCH = KC + 4, VW = 0;
  __device__ static int row(int kq, int q) { return 4 * kq + q; }
};

template <int P, int RB>
struct SlabLds {
  typedef SlabElem<P> E;
  static constexpr int XP = KC + E::VW;  // row pitch of a window
  typename E::in_t b[(P == PREC_BF16 ? 64 : KC) * E::PITCH];
  typename E::in_t x[NW][P == PREC_BF16 ? 8 : 16 * RB * XP];
  const typename E::in_t* xrow[NW][16 * RB];  // per wave: rows of the tile being loaded
  typename E::out_t* trow[NW][2][16 * RB];    // and the output rows of a tile and the next one
};

__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// rows [row0, row1) of the unit's stacked rows times its strip of columns
template <int P, int RB, int CB>
__device__ inline void slab_tile(const SlabUnit& u, const SlabJob* __restrict__ jobs, int wave, int lane,
                                 const typename SlabElem<P>::in_t* psi, SlabLds<P, RB>& lds) {
  typedef SlabElem<P> E;
  typedef typename E::in_t in_t;
  typedef typename E::out_t out_t;
  typedef typename E::acc_t acc_t;
  constexpr bool BF = P == PREC_BF16;
  constexpr int KG = E::KG, PITCH = E::PITCH, KW = KC, XP = SlabLds<P, RB>::XP;
  constexpr int LPR = BF ? 4 : KW / (E::VW > 0 ? E::VW : 1), RPI = 64 / LPR;  // lanes per row, rows per load
  constexpr int NL = BF ? RB * KW / KG : 16 * RB / RPI;                       // loads of a window
  const int r = lane & 15, kq = lane >> 4;
  const int gl = lane % LPR, sub = lane / LPR;
  const int tiles = (u.row1 - u.row0 + 16 * RB * NW - 1) / (16 * RB * NW);  // of each wave
  const int windows = (u.K + KW - 1) / KW;
  const bool whole = u.K <= KC;
  typedef __attribute__((address_space(1))) const in_t gin_t;
  typedef __attribute__((address_space(1))) out_t gout_t;
  in_t* const xw = lds.x[wave];

  // column of this lane in block j, blocks in pairs: 2 r and 2 r + 1 of 32 columns
  auto paired = [](int j) { return (j | 1) < CB; };
  auto col = [&](int j) { return 16 * (j & ~1) + (paired(j) ? 2 * r + (j & 1) : r); };

  auto stage = [&](int k0) {
    const int n = min(lane, u.N - 1);
    const bool cv = lane < u.N;
    const gin_t* B = (const gin_t*)psi + u.boff + n;
    constexpr int ST = KC / NW;  // rows of each wave, all in flight
    in_t v[ST];
#pragma unroll
    for (int i = 0; i < ST; ++i) {
      const int k = k0 + (BF ? 2 * (wave + i / 2 * NW) + (i & 1) : wave + i * NW);
      v[i] = k < u.K ? B[(long)min(k, u.K - 1) * u.ldb] : (in_t)0;
    }
    if (lane < 16 * CB) {
      if constexpr (BF) {
#pragma unroll
        for (int i = 0; i < ST; i += 2)
          *(uint32_t*)(lds.b + lane * PITCH + 2 * (wave + i / 2 * NW)) = cv ? v[i] | ((uint32_t)v[i + 1] << 16) : 0;
      } else {
#pragma unroll
        for (int i = 0; i < ST; ++i) lds.b[(wave + i * NW) * PITCH + lane] = cv ? v[i] : (in_t)0;
      }
    }
  };

  // matrix and row of tile row `lane` (rows past the last read it again)
  SlabJob jb;
  int m = 0;
  auto look = [&](int t) {
    const int row = min(u.row0 + (NW * t + wave) * 16 * RB + lane, u.row1 - 1);
    const int f = (unsigned)row / (unsigned)u.M;
    m = row - f * u.M;
    jb = jobs[u.job0 + f];
  };
  auto place = [&](int t) {
    int mm = m;
    asm volatile("" : "+v"(mm));  // computed here, not where the lookup has yet to arrive
    if (lane < 16 * RB) {
      lds.xrow[wave][lane] = (const in_t*)jb.X + (long)mm * u.K;
      lds.trow[wave][t & 1][lane] = (out_t*)jb.T + (long)mm * u.ldt + u.n0;
    }
    wave_fence();
  };
  auto xp = [&](int j) { return lds.xrow[wave][BF ? 16 * j + r : RPI * j + sub]; };

  uint32_t x[NL][4];  // the window in flight
  auto load = [&](int w) {
    if constexpr (BF) {
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        const int kk = KW * w + KG * (j / RB) + 4 * kq;
        const in_t* p = xp(j % RB) + (kk < u.K ? kk : 0);
        // an odd element: from the dword below
        const v3ua v = *(__attribute__((address_space(1))) const v3ua*)((uintptr_t)p & ~(uintptr_t)3);
        x[j][0] = v[0];
        x[j][1] = v[1];
        x[j][2] = v[2];
        x[j][3] = ((uintptr_t)p & 2) * 8;
      }
    } else {
      const int kk = KW * w + E::VW * gl;
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        const v4ua v = *(__attribute__((address_space(1))) const v4ua*)(xp(j) + (kk < u.K ? kk : 0));
        __builtin_memcpy(x[j], &v, 16);
      }
    }
  };
  auto stash = [&](int w) {
    const int nv = u.K - (KW * w + E::VW * gl);  // elements of this lane before the row's end
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      constexpr int VW = E::VW > 0 ? E::VW : 1;
      in_t y[VW];
      __builtin_memcpy(y, x[j], sizeof(y));
#pragma unroll
      for (int h = 0; h < VW; ++h) y[h] = h < nv ? y[h] : (in_t)0;
      __builtin_memcpy(__builtin_assume_aligned(xw + (RPI * j + sub) * XP + VW * gl, 16), y, sizeof(y));
    }
  };

  look(0);
  place(0);
  load(0);
  if (whole) {
    stage(0);
    __syncthreads();
  }
  for (int t = 0; t < tiles; ++t) {
    if (t + 1 < tiles) look(t + 1);
    acc_t acc[RB][CB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[i][j] = acc_t{};
    for (int w = 0; w < windows; ++w) {
      const int kb = KW * w & (KC - 1), left = u.K - KW * w;
      if (!whole && kb == 0) {  // every wave of the workgroup has the same tiles and windows
        __syncthreads();
        stage(KW * w);
        __syncthreads();
      }
      v4s xa[NL];
      if constexpr (BF) {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
          const uint32_t v[2] = {__builtin_amdgcn_alignbit(x[j][1], x[j][0], x[j][3]),
                                 __builtin_amdgcn_alignbit(x[j][2], x[j][1], x[j][3])};
          uint16_t h[4];
          __builtin_memcpy(h, v, 8);
#pragma unroll
          for (int q = 0; q < 4; ++q) xa[j][q] = (short)(KG * (j / RB) + 4 * kq + q < left ? h[q] : 0);
        }
      } else {
        stash(w);
        wave_fence();
      }
      if (w + 1 < windows) {
        load(w + 1);
      } else if (t + 1 < tiles) {
        place(t + 1);
        load(0);
      }
      if constexpr (BF) {
#pragma unroll
        for (int g = 0; g < KW / KG; ++g) {
          if (KG * g < left) {
            v4s b[CB];
#pragma unroll
            for (int j = 0; j < CB; ++j) __builtin_memcpy(&b[j], lds.b + col(j) * PITCH + kb + KG * g + 4 * kq, 8);
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
              for (int j = 0; j < CB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(xa[g * RB + i], b[j], acc[i][j], 0, 0, 0);
          }
        }
      } else {
#pragma unroll
        for (int g = 0; g < KW / KG; ++g) {
          if (KG * g < left) {
            const bool one = left - KG * g <= 4;  // a last group of at most four k's is one step
            const in_t* xr = xw + r * XP + KG * g + (one ? kq : 2 * kq);
            in_t a[RB][2];
#pragma unroll
            for (int i = 0; i < RB; ++i) {
              a[i][0] = xr[16 * i * XP];
              a[i][1] = xr[16 * i * XP + 1];
            }
            const in_t* bw = lds.b + (kb + KG * g + (one ? kq : 2 * kq)) * PITCH;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              if (h == 1 && one) break;
              in_t b[CB];
#pragma unroll
              for (int j = 0; j < CB; ++j) b[j] = bw[h * PITCH + col(j)];
#pragma unroll
              for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int i = 0; i < RB; ++i) acc[i][j] = E::mfma(a[i][h], b[j], acc[i][j]);
            }
          }
        }
        wave_fence();
      }
    }
    const int first = u.row0 + (NW * t + wave) * 16 * RB;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tr = 16 * i + E::row(kq, q);
        if (first + tr < u.row1) {
          gout_t* p = (gout_t*)lds.trow[wave][t & 1][tr];
#pragma unroll
          for (int j = 0; j < CB; ++j) {
            const int n = col(j);
            if (paired(j) && n + 1 < u.N) {
              if (j & 1) continue;
              const out_t o[2] = {acc[i][j][q], acc[i][j | 1][q]};
              if constexpr (sizeof(out_t) == 8) {
                v4ua v;
                __builtin_memcpy(&v, o, 16);
                *(__attribute__((address_space(1))) v4ua*)(p + n) = v;
              } else {
                v2ua v;
                __builtin_memcpy(&v, o, 8);
                *(__attribute__((address_space(1))) v2ua*)(p + n) = v;
              }
            } else if (n < u.N && !(paired(j) && (j & 1))) {
              p[n] = acc[i][j][q];
            }
          }
        }
      }
  }
}

// TAG only gives each instantiation its own kernel name, so profiles can tell
// launches apart.
template <int P, int RB, int TAG>
__global__ __launch_bounds__(64 * NW, RB == 1 ? 5 : 4) void gemm_slab(const SlabUnit* __restrict__ units,
                                                                     const SlabJob* __restrict__ jobs, const void* __restrict__ B) {
  __shared__ __align__(16) SlabLds<P, RB> lds;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const SlabUnit u = units[blockIdx.x];
  switch ((u.N + 15) / 16) {
    case 1: slab_tile<P, RB, 1>(u, jobs, wave, lane, (const typename SlabElem<P>::in_t*)B, lds); break;
    case 2: slab_tile<P, RB, 2>(u, jobs, wave, lane, (const typename SlabElem<P>::in_t*)B, lds); break;
    case 3: slab_tile<P, RB, 3>(u, jobs, wave, lane, (const typename SlabElem<P>::in_t*)B, lds); break;
    default: slab_tile<P, RB, 4>(u, jobs, wave, lane, (const typename SlabElem<P>::in_t*)B, lds); break;
  }
}

template <int P, int TAG>
void launch(bool tall, const SlabUnit* units, int n_units, const SlabJob* jobs, const void* B, hipStream_t s) {
  if (tall) gemm_slab<P, 2, TAG><<<n_units, 64 * NW, 0, s>>>(units, jobs, B);
  else gemm_slab<P, 1, TAG><<<n_units, 64 * NW, 0, s>>>(units, jobs, B);
}

}  // namespace

void launch_gemm_slab(int prec, int tag, bool tall, const SlabUnit* units, int n_units, const SlabJob* jobs,
                      const void* B, hipStream_t s) {
  if (n_units <= 0) return;
  if (prec == PREC_F64 && tag == 3) launch<PREC_F64, 3>(tall, units, n_units, jobs, B, s);
  else if (prec == PREC_F64) launch<PREC_F64, 1>(tall, units, n_units, jobs, B, s);
  else if (prec == PREC_F32) launch<PREC_F32, 0>(tall, units, n_units, jobs, B, s);
  else launch<PREC_BF16, 0>(tall, units, n_units, jobs, B, s);
}

}  // namespace dmrg
