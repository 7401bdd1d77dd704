// Stream kernel: long lists of small block products, C = sum_j c_j A_j B_j^T
// (sigma phase B, fp64 and fp32), one wave per unit.
//
// What bounds the phase is bringing millions of small operands on chip: at
// CAS(20,20), M = 1024, 3.6 million items of mean K 12 (half of them K <= 4) in
// 1444 blocks of at most 62 x 62 read 22 GB of operands for 1.1e11 flops.  Taken
// one item at a time, each costs a round trip to memory and a barrier.  Here each
// wave owns a whole tile of an output block (up to 64 x 64, so every operand is
// read once per unit) and treats its items as one stream of segments of two elements:
//
//  * A window is SL consecutive segments of the stream, of whatever items; lane
//    (sub, g) loads segment g of rows sub, sub + 64 / SL, ...: SL lanes read a
//    contiguous stretch of a row.  (Loading the MFMA layout directly, 16 rows per
//    16 lanes, took 50 L1 accesses per load; this takes 25.)
//  * The window goes through the wave's own LDS into the MFMA layout; row
//    pitch KW + VW keeps both directions free of bank conflicts.  Nothing is
//    shared between waves: no barriers, no idle waves when a block is narrow.
//  * While a window is multiplied, the next window's operands and the one after
//    next's descriptors are in flight, across item boundaries.  SL is chosen so
//    that a window holds 10..16 KB for every tile.
//  * Segment g's item: a prefix sum of the next SL items' segment counts, the
//    start positions as a bit mask, and the count of start bits up to g.
//  * Rows past M (columns past N) read the last one again; their results are not
//    stored (partial tiles hold them, the reduction skips them).  Elements past an
//    item's K are read (DevMem keeps 64 readable bytes past every buffer) and
//    replaced by zeros in both operands.
//
// Sigma at CAS(20,20), M = 1024: 10.4 -> 8.3 ms (this kernel 7.5 -> 4.9 ms, now
// bound by 7.5 TB/s of L2 misses: without the MFMAs it takes 4.8 ms); CAS(12,12),
// M = 512: 1.80 -> 1.51 ms; CAS(8,8), M = 60: 192 -> 57 us; fp32, CAS(16,16),
// M = 512: 1.73 -> 1.15 ms, the same bits.  64-byte-wide windows (SL = 4) took 6.3 ms.
#include <hip/hip_runtime.h>

#include <stdexcept>

#include "kernels.hpp"

namespace dmrg {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v4ua __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int v2ua __attribute__((ext_vector_type(2), aligned(4)));

// one segment (VW elements) from global memory
template <typename T, int VW>
__device__ inline void load_segment(const char* p, T* x) {
  if constexpr (VW * sizeof(T) == 16) {
    const v4ua v = *(__attribute__((address_space(1))) const v4ua*)p;
    __builtin_memcpy(x, &v, 16);
  } else {
    const v2ua v = *(__attribute__((address_space(1))) const v2ua*)p;
    __builtin_memcpy(x, &v, 8);
  }
}

template <typename T>
struct Elem;
// VW: elements of a segment (one lane's load); SG: an item starts at a segment
// that is a multiple of SG and is filled up with zeros to the next one.  fp64
// packs items segment by segment; fp32 keeps the k grouping of the fp32 MFMA (8
// k's of one item, even ones first), so that its rounding does not depend on
// which items share a window.
template <>
struct Elem<double> {
  static constexpr int VW = 2, SG = 1;
  typedef v4d acc_t;
  __device__ static acc_t mfma(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int kq, int q) { return kq + 4 * q; }  // accumulator element q of lane group kq
};
template <>
struct Elem<float> {
  static constexpr int VW = 2, SG = 4;
  typedef v4f acc_t;
  __device__ static acc_t mfma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int kq, int q) { return 4 * kq + q; }
};

// lane l <- lane l - D of its row of 16 (callers discard lanes without a source)
template <int D>
__device__ inline int row_shr(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x110 + D, 0xf, 0xf, false);
}
template <int D>
__device__ inline int row_ror(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x120 + D, 0xf, 0xf, false);
}

constexpr int kWaveLds = 128 * 18 * 8;  // bytes of LDS per wave (128 rows of 16 doubles, 16 bytes of padding each)

template <typename T, int RB, int CB, int SL>
__device__ inline void stream_tile(const GemmUnit& u, const GemmItem* __restrict__ items, int lane, T* lds) {
  typedef Elem<T> E;
  typedef typename E::acc_t acc_t;
  constexpr int VW = E::VW, SG = E::SG, SB = VW * (int)sizeof(T);  // segment bytes
  constexpr int KW = SL * VW, PITCH = KW + VW, RPI = 64 / SL;
  constexpr int NA = 16 * RB / RPI, NB = 16 * CB / RPI, LB = 16 / RPI;  // loads; loads of one 16-row block
  static_assert((16 * RB + 16 * CB) * PITCH * (int)sizeof(T) <= kWaveLds, "window larger than the wave's LDS");
  const int g = lane & (SL - 1), sub = lane / SL;
  const int r = lane & 15, kq = lane >> 4;
  acc_t acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = acc_t{};

  // depths of items kb + lane and kb + 64 + lane
  int kb = u.ib;
  auto depth_of = [&](int i) { return items[min(i, u.ie - 1)].K; };
  int ka = depth_of(kb + lane), kc = depth_of(kb + 64 + lane);
  int it0 = u.ib, s0 = 0;  // next segment: segment s0 of item it0

  // next window: this lane's item and first k, and the window's segments
  int ix = 0, kk = 0, nseg = 0;
  auto plan = [&]() {
    const int j = it0 - kb + g;
    const int x = __builtin_amdgcn_ds_bpermute((j & 63) * 4, ka), y = __builtin_amdgcn_ds_bpermute((j & 63) * 4, kc);
    const int K = it0 + g < u.ie ? (j < 64 ? x : y) : 0;
    const int ns = (K + VW * SG - 1) / (VW * SG) * SG - (g == 0 ? s0 : 0);
    int P = ns, t;
    t = row_shr<1>(P);
    P += g >= 1 ? t : 0;
    t = row_shr<2>(P);
    P += g >= 2 ? t : 0;
    if constexpr (SL >= 8) {
      t = row_shr<4>(P);
      P += g >= 4 ? t : 0;
    }
    if constexpr (SL >= 16) {
      t = row_shr<8>(P);
      P += (g & 15) >= 8 ? t : 0;
    }
    if constexpr (SL == 32) {
      t = __builtin_amdgcn_readlane(P, 15);
      P += g >= 16 ? t : 0;
    }
    const int first = P - ns;  // window segment the item starts at
    int m = ns > 0 && first < SL ? (int)(1u << first) : 0;
    m |= row_ror<1>(m);
    m |= row_ror<2>(m);
    if constexpr (SL >= 8) m |= row_ror<4>(m);
    if constexpr (SL >= 16) m |= row_ror<8>(m);
    unsigned starts = __builtin_amdgcn_readlane(m, 0);
    if constexpr (SL == 32) starts |= __builtin_amdgcn_readlane(m, 16);
    const int total = __builtin_amdgcn_readlane(P, SL - 1);
    const bool whole = __builtin_amdgcn_ballot_w64(ns > 0 && P == SL) != 0;  // an item ends with the window
    nseg = min(total, SL);
    const unsigned low = starts & ((2u << g) - 1u);
    const int idx = __builtin_popcount(low) - 1;
    const int off = g - (31 - __builtin_clz(low | 1u)) + (idx <= 0 ? s0 : 0);
    ix = g < nseg ? it0 + idx : u.ie - 1;
    kk = g < nseg ? off * VW : 0;  // past K where SG > 1 fills up: read at 0, see load
    if (total < SL) {
      it0 = u.ie;
      s0 = 0;
    } else {
      const int il = __builtin_popcount(starts) - 1;
      const int ol = SL - 1 - (31 - __builtin_clz(starts | 1u)) + (il <= 0 ? s0 : 0);
      it0 += whole ? il + 1 : il;
      s0 = whole ? 0 : ol + 1;
    }
    if (it0 - kb >= 64) {
      kb += 64;
      ka = kc;
      kc = depth_of(kb + 64 + lane);
    }
  };
  // descriptor of this lane's item
  GemmItem d;
  T xa[NA][VW], xb[NB][VW];  // the window's operands in flight
  T cf = (T)0;
  int nv = 0;  // valid elements of this lane's segment
  auto load = [&](int n) {
    nv = g < n ? max(min(VW, d.K - kk), 0) : 0;
    cf = (T)d.coef;
    if (nv == 0) kk = 0;
    // rows m0 + sub + RPI j; those past the last one read it again (never stored)
    const int la = u.M - 1 - u.m0 - sub, lb = u.N - 1 - u.n0 - sub;  // row steps left
    const char* pa = (const char*)d.A + ((long)(u.m0 + sub + min(la, 0)) * d.lda + kk) * (long)sizeof(T);
    const char* pb = (const char*)d.B + ((long)(u.n0 + sub + min(lb, 0)) * d.ldb + kk) * (long)sizeof(T);
    const int sa = d.lda * (int)sizeof(T), sb = d.ldb * (int)sizeof(T);
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const int st = j < NA - LB ? RPI * j : max(min(RPI * j, la), 0);
      load_segment<T, VW>(pa + (long)st * sa, xa[j]);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int st = j < NB - LB ? RPI * j : max(min(RPI * j, lb), 0);
      load_segment<T, VW>(pb + (long)st * sb, xb[j]);
    }
  };
  auto stash = [&]() {
    T* w = lds + sub * PITCH + g * VW;
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      T y[VW];
#pragma unroll
      for (int h = 0; h < VW; ++h) y[h] = h < nv ? xa[j][h] * cf : (T)0;
      __builtin_memcpy(__builtin_assume_aligned(w + RPI * j * PITCH, SB), y, SB);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      T y[VW];
#pragma unroll
      for (int h = 0; h < VW; ++h) y[h] = h < nv ? xb[j][h] : (T)0;
      __builtin_memcpy(__builtin_assume_aligned(w + (16 * RB + RPI * j) * PITCH, SB), y, SB);
    }
  };
  if (u.ib < u.ie) {
    plan();
    d = items[ix];
    int now = nseg;
    load(now);
    plan();
    d = items[ix];
    while (now > 0) {
      stash();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int nxt = nseg;
      if (nxt > 0) {
        load(nxt);
        nseg = 0;
        if (it0 < u.ie) {
          plan();
          d = items[ix];
        }
      }
#pragma unroll
      for (int q = 0; q < SL / 4; ++q) {
        if (4 * q < now) {
          T a[RB][VW], b[CB][VW];
#pragma unroll
          for (int i = 0; i < RB; ++i)
            __builtin_memcpy(a[i], __builtin_assume_aligned(lds + (16 * i + r) * PITCH + (4 * q + kq) * VW, SB), SB);
#pragma unroll
          for (int j = 0; j < CB; ++j)
            __builtin_memcpy(b[j], __builtin_assume_aligned(lds + (16 * (RB + j) + r) * PITCH + (4 * q + kq) * VW, SB), SB);
#pragma unroll
          for (int h = 0; h < VW; ++h)
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
              for (int i = 0; i < RB; ++i) acc[i][j] = E::mfma(a[i][h], b[j][h], acc[i][j]);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      now = nxt;
    }
  }
  T* C = (T*)u.C;
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tr = 16 * i + E::row(kq, q), tc = 16 * j + r;
        const int gm = u.m0 + tr, gn = u.n0 + tc;
        const T v = acc[i][j][q];
        if (u.accumulate == 2) {
          C[tr * (16 * CB) + tc] = v;  // partial slot, full tile
        } else if (gm < u.M && gn < u.N) {
          const long idx = (long)gm * u.ldc + gn;
          C[idx] = u.accumulate ? C[idx] + v : v;
        }
      }
}

// segments per row of a window: 128 bytes of a row for the large tiles, more for
// the small ones (about 16 KB of operands in flight per wave for every tile)
template <typename T>
constexpr int window_segments(int rb, int cb) {
  const int s = rb + cb >= 5 ? 128 : (rb + cb >= 3 ? 256 : 512);
  const int n = s / (Elem<T>::VW * (int)sizeof(T));
  return n > 32 ? 32 : n;
}

template <typename T, int RB>
__device__ inline void stream_row(const GemmUnit& u, const GemmItem* __restrict__ items, int lane, T* lds) {
  switch (u.shape & 7) {
    case 1: stream_tile<T, RB, 1, window_segments<T>(RB, 1)>(u, items, lane, lds); break;
    case 2: stream_tile<T, RB, 2, window_segments<T>(RB, 2)>(u, items, lane, lds); break;
    case 3: stream_tile<T, RB, 3, window_segments<T>(RB, 3)>(u, items, lane, lds); break;
    default: stream_tile<T, RB, 4, window_segments<T>(RB, 4)>(u, items, lane, lds); break;
  }
}

template <typename T, int TAG>
__global__ __launch_bounds__(256, 2) void gemm_stream(const GemmUnit* __restrict__ units,
                                                      const GemmItem* __restrict__ items, int n_units) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  __shared__ __align__(16) char mem[4][kWaveLds];
  T* lds = reinterpret_cast<T*>(mem[wave]);
  const int ui = blockIdx.x * 4 + wave;
  if (ui >= n_units) return;  // whole wave exits; the kernel has no barriers
  const GemmUnit u = units[ui];
  switch (u.shape >> 3) {
    case 1: stream_row<T, 1>(u, items, lane, lds); break;
    case 2: stream_row<T, 2>(u, items, lane, lds); break;
    case 3: stream_row<T, 3>(u, items, lane, lds); break;
    default: stream_row<T, 4>(u, items, lane, lds); break;
  }
}

}  // namespace

void launch_gemm_stream(int prec, int tag, const GemmUnit* units, int n_units, const GemmItem* items, hipStream_t s) {
  if (n_units <= 0) return;
  const dim3 grid((n_units + 3) / 4), blk(256);
  if (prec == PREC_F32) gemm_stream<float, 0><<<grid, blk, 0, s>>>(units, items, n_units);
  else if (tag == 2) gemm_stream<double, 2><<<grid, blk, 0, s>>>(units, items, n_units);
  else if (tag == 4) gemm_stream<double, 4><<<grid, blk, 0, s>>>(units, items, n_units);
  else gemm_stream<double, 0><<<grid, blk, 0, s>>>(units, items, n_units);
}

}  // namespace dmrg
