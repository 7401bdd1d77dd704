// Stream kernel: long lists of small block products, C = sum_j c_j A_j B_j^T
// (sigma phase B), one wave per unit.
//
// What bounds the phase is bringing millions of small operands on chip: at
// CAS(20,20), M = 1024, 3.6 million items of mean K 12 (half of them K <= 4) in
// 1444 blocks of at most 62 x 62 read 22 GB of operands for 1.1e11 flops.  Taken
// one item at a time, each costs a round trip to memory and a barrier.  Here each
// wave owns a whole tile of an output block (up to 64 x 64, so every operand is
// read once per unit) and treats its items as one stream of segments (two k's; bf16 four):
//
//  * A window is SL consecutive segments of the stream, of whatever items; lane
//    (sub, g) loads segment g of rows sub, sub + 64 / SL, ...: SL lanes read a
//    contiguous stretch of a row.  (Loading the MFMA layout directly, 16 rows per
//    16 lanes, took 50 L1 accesses per load; this takes 25.)
//  * The window goes through the wave's own LDS into the MFMA layout; a row
//    pitch of SL + 1 segments keeps both directions free of bank conflicts.  Nothing is
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
// This kernel on a random state (mean K 12) of CAS(20,20), M = 1024, against the
// workgroup kernel of up to 96 x 64 before it: 7.5 -> 5.20 ms (37 GB of L2 misses;
// without the MFMAs 4.8 ms, with A from one place 2.8); on the state of a half sweep
// there (mean K 23, blocks of up to 82 x 62) 5.46 -> 5.37 ms (39 GB, where that kernel,
// whose waves shared A, missed 25).  CAS(12,12), M = 512: 1.36 -> 1.07 ms; CAS(16,16),
// M = 512, with the bits of the kernels before: fp32 1.34 -> 0.82 ms, bf16 0.94 -> 0.75
// ms.  64-byte-wide windows (SL = 4) took 6.3 ms in fp64.
#include <hip/hip_runtime.h>

#include "bf16.hpp"
#include "kernels.hpp"

namespace dmrg {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef unsigned int v4ua __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int v3ua __attribute__((ext_vector_type(3), aligned(4)));
typedef unsigned int v2ua __attribute__((ext_vector_type(2), aligned(4)));

// VW: k's of a segment (one lane's load of a row); SG: an item starts at a segment
// that is a multiple of SG and is filled up with zeros to the next one.  fp64
// packs items segment by segment; fp32 and bf16 keep the k grouping of their MFMAs
// (8 k's of one item, even ones first; 16 k's of one item), so that their rounding
// does not depend on which items share a window.  A segment of A or B in memory,
// as loaded (RawA, RawB), and in LDS (Seg, of which an item's first nv k's count).
template <int P>
struct Elem;
template <>
struct Elem<PREC_F64> {
  typedef double ta;
  typedef double tb;
  typedef double out_t;
  typedef v4d acc_t;
  static constexpr int VW = 2, SG = 1, STEPS = 2;
  struct Seg { double x[2]; };
  typedef Seg RawA;
  typedef Seg RawB;
  __device__ static Seg load(const char* p) {
    const v4ua v = *(__attribute__((address_space(1))) const v4ua*)p;
    Seg y;
    __builtin_memcpy(&y, &v, 16);
    return y;
  }
  __device__ static RawA load_a(const char* p) { return load(p); }
  __device__ static RawB load_b(const char* p) { return load(p); }
  __device__ static Seg seg_a(const RawA& v, double c, int nv) {
    return {{0 < nv ? v.x[0] * c : 0.0, 1 < nv ? v.x[1] * c : 0.0}};
  }
  __device__ static Seg seg_b(const RawB& v, int nv) { return {{0 < nv ? v.x[0] : 0.0, 1 < nv ? v.x[1] : 0.0}}; }
  __device__ static acc_t mfma(const Seg& a, const Seg& b, int h, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a.x[h], b.x[h], c, 0, 0, 0);
  }
  __device__ static int row(int kq, int q) { return kq + 4 * q; }  // accumulator element q of lane group kq
};
template <>
struct Elem<PREC_F32> {
  typedef float ta;
  typedef float tb;
  typedef float out_t;
  typedef v4f acc_t;
  static constexpr int VW = 2, SG = 4, STEPS = 2;
  struct Seg { float x[2]; };
  typedef Seg RawA;
  typedef Seg RawB;
  __device__ static Seg load(const char* p) {
    const v2ua v = *(__attribute__((address_space(1))) const v2ua*)p;
    Seg y;
    __builtin_memcpy(&y, &v, 8);
    return y;
  }
  __device__ static RawA load_a(const char* p) { return load(p); }
  __device__ static RawB load_b(const char* p) { return load(p); }
  __device__ static Seg seg_a(const RawA& v, float c, int nv) {
    return {{0 < nv ? v.x[0] * c : 0.f, 1 < nv ? v.x[1] * c : 0.f}};
  }
  __device__ static Seg seg_b(const RawB& v, int nv) { return {{0 < nv ? v.x[0] : 0.f, 1 < nv ? v.x[1] : 0.f}}; }
  __device__ static acc_t mfma(const Seg& a, const Seg& b, int h, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[h], b.x[h], c, 0, 0, 0);
  }
  __device__ static int row(int kq, int q) { return 4 * kq + q; }
};
template <>
struct Elem<PREC_BF16_A32> {
  typedef float ta;
  typedef uint16_t tb;
  typedef float out_t;
  typedef v4f acc_t;
  static constexpr int VW = 4, SG = 4, STEPS = 1;
  struct Seg { v4s x; };
  struct RawA { v4ua v; };
  struct RawB { v3ua v; unsigned sh; };  // from the dword at or below the first k; bits to drop
  __device__ static RawA load_a(const char* p) { return {*(__attribute__((address_space(1))) const v4ua*)p}; }
  __device__ static RawB load_b(const char* p) {
    return {*(__attribute__((address_space(1))) const v3ua*)((uintptr_t)p & ~(uintptr_t)3), (unsigned)((uintptr_t)p & 2) * 8};
  }
  __device__ static Seg seg_a(const RawA& v, float c, int nv) {
    Seg y;
#pragma unroll
    for (int h = 0; h < 4; ++h) y.x[h] = (short)(h < nv ? f2bf(__uint_as_float(v.v[h]) * c) : 0);
    return y;
  }
  __device__ static Seg seg_b(const RawB& v, int nv) {
    const uint32_t w[2] = {__builtin_amdgcn_alignbit(v.v[1], v.v[0], v.sh), __builtin_amdgcn_alignbit(v.v[2], v.v[1], v.sh)};
    Seg y;
    __builtin_memcpy(&y, w, 8);
#pragma unroll
    for (int h = 0; h < 4; ++h) y.x[h] = (short)(h < nv ? y.x[h] : 0);
    return y;
  }
  __device__ static acc_t mfma(const Seg& a, const Seg& b, int, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.x, b.x, c, 0, 0, 0);
  }
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

template <int P, int RB, int CB, int SL>
__device__ inline void stream_tile(const GemmUnit& u, const GemmItem* __restrict__ items, int lane, char* mem) {
  typedef Elem<P> E;
  typedef typename E::acc_t acc_t;
  typedef typename E::out_t out_t;
  typedef typename E::Seg Seg;
  constexpr int VW = E::VW, SG = E::SG;
  constexpr int PITCH = SL + 1, RPI = 64 / SL;  // segments per row of the window in LDS, rows per load
  constexpr int NA = 16 * RB / RPI, NB = 16 * CB / RPI, LB = 16 / RPI;  // loads; loads of one 16-row block
  static_assert((16 * RB + 16 * CB) * PITCH * (int)sizeof(Seg) <= kWaveLds, "window larger than the wave's LDS");
  Seg* const lds = reinterpret_cast<Seg*>(mem);
  const int g = lane & (SL - 1), sub = lane / SL;
  const int r = lane & 15, kq = lane >> 4;
  acc_t acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = acc_t{};

  // depths of items kb + lane and kb + 64 + lane
  int kb = u.ib;
  auto depth_of = [&](int i) { return list_depth(items, i, u.ib, u.ie); };
  int ka = depth_of(kb + lane), kc = depth_of(kb + 64 + lane);
  int it0 = u.ib, s0 = 0;  // next segment: segment s0 of item it0

  // next window: this lane's item and first k, and the window's segments
  int ix = 0, kk = 0, nseg = 0;
  auto plan = [&]() {
    const int j = it0 - kb + g;
    const int x = __builtin_amdgcn_ds_bpermute((j & 63) * 4, ka), y = __builtin_amdgcn_ds_bpermute((j & 63) * 4, kc);
    const int K = it0 + g < u.ie ? (j < 64 ? x : y) : 0;
    const int ns = (K + VW * SG - 1) / (VW * SG) * SG - (g == 0 ? s0 : 0);
    int sum = ns, t;
    t = row_shr<1>(sum);
    sum += g >= 1 ? t : 0;
    t = row_shr<2>(sum);
    sum += g >= 2 ? t : 0;
    if constexpr (SL >= 8) {
      t = row_shr<4>(sum);
      sum += g >= 4 ? t : 0;
    }
    if constexpr (SL >= 16) {
      t = row_shr<8>(sum);
      sum += (g & 15) >= 8 ? t : 0;
    }
    if constexpr (SL == 32) {
      t = __builtin_amdgcn_readlane(sum, 15);
      sum += g >= 16 ? t : 0;
    }
    const int first = sum - ns;  // window segment the item starts at
    int m = ns > 0 && first < SL ? (int)(1u << first) : 0;
    m |= row_ror<1>(m);
    m |= row_ror<2>(m);
    if constexpr (SL >= 8) m |= row_ror<4>(m);
    if constexpr (SL >= 16) m |= row_ror<8>(m);
    unsigned starts = __builtin_amdgcn_readlane(m, 0);
    if constexpr (SL == 32) starts |= __builtin_amdgcn_readlane(m, 16);
    const int total = __builtin_amdgcn_readlane(sum, SL - 1);
    const bool whole = __builtin_amdgcn_ballot_w64(ns > 0 && sum == SL) != 0;  // an item ends with the window
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
  typename E::RawA xa[NA];  // the window's operands in flight
  typename E::RawB xb[NB];
  out_t cf = (out_t)0;
  int nv = 0;  // valid elements of this lane's segment
  auto load = [&](int n) {
    nv = g < n ? max(min(VW, d.K - kk), 0) : 0;
    cf = (out_t)d.coef;
    if (nv == 0) kk = 0;
    // rows m0 + sub + RPI j; those past the last one read it again (never stored)
    const int la = u.M - 1 - u.m0 - sub, lb = u.N - 1 - u.n0 - sub;  // row steps left
    const char* pa = (const char*)d.A + ((long)(u.m0 + sub + min(la, 0)) * d.lda + kk) * (long)sizeof(typename E::ta);
    const char* pb = (const char*)d.B + ((long)(u.n0 + sub + min(lb, 0)) * d.ldb + kk) * (long)sizeof(typename E::tb);
    const int sa = d.lda * (int)sizeof(typename E::ta), sb = d.ldb * (int)sizeof(typename E::tb);
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const int st = j < NA - LB ? RPI * j : max(min(RPI * j, la), 0);
      xa[j] = E::load_a(pa + (long)st * sa);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int st = j < NB - LB ? RPI * j : max(min(RPI * j, lb), 0);
      xb[j] = E::load_b(pb + (long)st * sb);
    }
  };
  auto stash = [&]() {
    Seg* w = lds + sub * PITCH + g;
#pragma unroll
    for (int j = 0; j < NA; ++j) w[RPI * j * PITCH] = E::seg_a(xa[j], cf, nv);
#pragma unroll
    for (int j = 0; j < NB; ++j) w[(16 * RB + RPI * j) * PITCH] = E::seg_b(xb[j], nv);
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
          Seg a[RB], b[CB];
#pragma unroll
          for (int i = 0; i < RB; ++i) a[i] = lds[(16 * i + r) * PITCH + 4 * q + kq];
#pragma unroll
          for (int j = 0; j < CB; ++j) b[j] = lds[(16 * (RB + j) + r) * PITCH + 4 * q + kq];
#pragma unroll
          for (int h = 0; h < E::STEPS; ++h)
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
              for (int i = 0; i < RB; ++i) acc[i][j] = E::mfma(a[i], b[j], h, acc[i][j]);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      now = nxt;
    }
  }
  out_t* C = (out_t*)u.C;
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tr = 16 * i + E::row(kq, q), tc = 16 * j + r;
        const int gm = u.m0 + tr, gn = u.n0 + tc;
        const out_t v = acc[i][j][q];
        if (u.accumulate == 2) {
          C[tr * (16 * CB) + tc] = v;  // partial slot, full tile
        } else if (gm < u.M && gn < u.N) {
          const long idx = (long)gm * u.ldc + gn;
          C[idx] = u.accumulate ? C[idx] + v : v;
        }
      }
}

// segments per row of a window: 128 bytes of a row of A for the large tiles, more for
// the small ones (about 16 KB of operands in flight per wave for every tile); bf16,
// whose items take 16 k's however shallow they are, twice that (four items of a 64 x 64
// tile instead of two: 836 -> 764 us at CAS(16,16), M = 512)
template <int P>
constexpr int window_segments(int rb, int cb) {
  const int s = (rb + cb >= 5 ? 128 : (rb + cb >= 3 ? 256 : 512)) * (P == PREC_BF16_A32 ? 2 : 1);
  const int n = s / (Elem<P>::VW * (int)sizeof(typename Elem<P>::ta));
  return n > 32 ? 32 : n;
}

template <int P, int RB>
__device__ inline void stream_row(const GemmUnit& u, const GemmItem* __restrict__ items, int lane, char* lds) {
  switch (u.shape & 7) {
    case 1: stream_tile<P, RB, 1, window_segments<P>(RB, 1)>(u, items, lane, lds); break;
    case 2: stream_tile<P, RB, 2, window_segments<P>(RB, 2)>(u, items, lane, lds); break;
    case 3: stream_tile<P, RB, 3, window_segments<P>(RB, 3)>(u, items, lane, lds); break;
    default: stream_tile<P, RB, 4, window_segments<P>(RB, 4)>(u, items, lane, lds); break;
  }
}

template <int P, int TAG>
__global__ __launch_bounds__(256, 2) void gemm_stream(const GemmUnit* __restrict__ units,
                                                      const GemmItem* __restrict__ items, int n_units) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  __shared__ __align__(16) char mem[4][kWaveLds];
  const int ui = blockIdx.x * 4 + wave;
  if (ui >= n_units) return;  // whole wave exits; the kernel has no barriers
  const GemmUnit u = units[ui];
  switch (u.shape >> 3) {
    case 1: stream_row<P, 1>(u, items, lane, mem[wave]); break;
    case 2: stream_row<P, 2>(u, items, lane, mem[wave]); break;
    case 3: stream_row<P, 3>(u, items, lane, mem[wave]); break;
    default: stream_row<P, 4>(u, items, lane, mem[wave]); break;
  }
}

}  // namespace

void launch_gemm_stream(int prec, int tag, const GemmUnit* units, int n_units, const GemmItem* items, hipStream_t s) {
  if (n_units <= 0) return;
  const dim3 grid((n_units + 3) / 4), blk(256);
  if (prec == PREC_F32) gemm_stream<PREC_F32, 0><<<grid, blk, 0, s>>>(units, items, n_units);
  else if (prec == PREC_BF16_A32) gemm_stream<PREC_BF16_A32, 0><<<grid, blk, 0, s>>>(units, items, n_units);
  else if (tag == 2) gemm_stream<PREC_F64, 2><<<grid, blk, 0, s>>>(units, items, n_units);
  else if (tag == 4) gemm_stream<PREC_F64, 4><<<grid, blk, 0, s>>>(units, items, n_units);
  else gemm_stream<PREC_F64, 0><<<grid, blk, 0, s>>>(units, items, n_units);
}

}  // namespace dmrg
