// fp32 products on the 16-bit matrix cores: every fp32 operand is split into
// 16-bit pieces as it is staged in LDS, and a product is formed from the
// products of the pieces in fp32 accumulators.  Two formats:
//
//   kF16x2  x 2^s = h + l, two fp16 pieces (11 + 11 bits; a power of two
//           brings the operand's largest value near 2^14, so that l keeps its
//           11 bits down to 2^-17 of it and an absolute 2^-39 of it below);
//           a b = h h + h l + l h: three v_mfma_f32_32x32x16_f16.  Left out
//           and rounded away: 2^-23.5 rms of |a b|, of either sign.
//   kBf16x3 x = h + m + l exactly, three bf16 pieces (8 + 8 + 8 bits, the
//           range of fp32: no scale); a b = hh + hm + mh + hl + lh + mm: six
//           v_mfma_f32_32x32x16_bf16.  Left out: 2^-24.5 rms.
//   kBf16   x rounded to one bf16 (the bf16 selection mode, not a split).
//
// Why: under sustained load with random data the fp32 MFMA
// (v_mfma_f32_32x32x2_f32) gives 107-120 TFLOP/s on this chip, the bf16 one
// 1510 and the fp16 one 1440 (loops over registers): 252 and 480 TFLOP/s of
// products.  The accumulators of a matrix instruction round more often than
// one fp32 addition per instruction would (measured: a contraction of 4096
// through one accumulator was 1.9 times as far from 64 bits as the fp32
// MFMA's), so the accumulators are added into a second set every
// kSplitFlush slices and cleared: the sums that are rounded stay short.
#pragma once

#include "glr_device.hpp"

namespace glr {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// two floats rounded to bf16 (nearest even), the first in the low half
__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

enum SplitFmt { kF16x2, kBf16x3, kBf16 };
constexpr int split_pieces(SplitFmt f) { return f == kF16x2 ? 2 : f == kBf16x3 ? 3 : 1; }

// The pieces of two floats, packed by piece (the first value in the low half).
// kBf16x3: h is x truncated (rounding it could overflow), m the rounded
// remainder, l what is left (exact: 8 bits).
template <SplitFmt F>
__device__ __forceinline__ void split_pair(float x0, float x1, float scale, uint32_t (&p)[split_pieces(F)]) {
  if constexpr (F == kF16x2) {
    const float y0 = x0 * scale, y1 = x1 * scale;
    const f16x2 h = __builtin_convertvector(f32x2{y0, y1}, f16x2);
    const f16x2 l = __builtin_convertvector(
        f32x2{__builtin_fmaf((float)h[0], -1.0f, y0), __builtin_fmaf((float)h[1], -1.0f, y1)}, f16x2);
    p[0] = __builtin_bit_cast(uint32_t, h);
    p[1] = __builtin_bit_cast(uint32_t, l);
  } else if constexpr (F == kBf16x3) {
    const uint32_t u0 = __float_as_uint(x0), u1 = __float_as_uint(x1);
    p[0] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);   // the upper halves
    const float r0 = x0 - __uint_as_float(u0 & 0xFFFF0000u), r1 = x1 - __uint_as_float(u1 & 0xFFFF0000u);
    p[1] = pk_bf16(r0, r1);
    const float s0 = r0 - __uint_as_float(p[1] << 16), s1 = r1 - __uint_as_float(p[1] & 0xFFFF0000u);
    p[2] = pk_bf16(s0, s1);
  } else {
    p[0] = pk_bf16(x0, x1);
  }
}
template <SplitFmt F>
__device__ __forceinline__ f32x16 split_mfma(u32x4 a, u32x4 b, f32x16 c) {
  if constexpr (F == kF16x2)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
  else
    return mfma32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c);
}
// the power of two that brings amax into [2^14, 2^15), as an exponent (0 for
// an all-zero or non-finite operand)
__device__ __forceinline__ int split_exp(float amax) {
  if (!(amax > 0.f) || !isfinite(amax)) return 0;
  const int e = 14 - ilogbf(amax);
  return e < 126 ? e : 126;
}

// Where an operand's scale comes from (kF16x2): the exponent `fixed`, or with
// `amax` the one of the largest of n partial maxima times `mul` (a bound on
// the operand's largest value), at most `cap` (`fixed` when they are all zero).
// `basis`: the bound is for an orthonormal basis of the product, and *basis the
// largest entry of the one taken.
struct SplitScale {
  const float* amax;
  int n;
  float mul;
  int fixed;
  int cap = 127;
  const float* basis = nullptr;
};
// rows of an orthonormal basis: |u| <= 1, with room for a basis that is not
// quite one (fp16 ends at 2^16)
constexpr int kUnitExp = 6;
inline SplitScale split_unit() { return {nullptr, 0, 1.f, kUnitExp}; }
// rows of a basis that a caller may have written: *umax its largest entry, 0
// when the library computed it
inline SplitScale split_basis(const float* umax) { return {umax, 1, 1.f, kUnitExp, kUnitExp}; }
__device__ __forceinline__ int split_basis_exp(float umax) {
  if (!(umax > 0.f)) return kUnitExp;
  const int e = split_exp(umax);
  return e < kUnitExp ? e : kUnitExp;
}
// the exponent, by a whole workgroup (red: one float per wave)
__device__ __forceinline__ int split_block_exp(const SplitScale& sc, float* red) {
  if (!sc.amax) return sc.fixed;
  float mx = 0.f;
  for (int i = threadIdx.x; i < sc.n; i += kThreads) mx = fmaxf(mx, sc.amax[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (lane_id() == 0) red[wave_id()] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])) * sc.mul;
  __syncthreads();
  if (sc.basis && *sc.basis > 1.5f) mx *= *sc.basis * sc.mul;   // (its rows' norms: mul is sqrt(d))
  if (mx == 0.f) return sc.fixed;
  const int e = split_exp(mx);
  return e < sc.cap ? e : sc.cap;
}

// A slice of one operand in LDS: PIECES planes of R rows (the operand's M or
// N index) of kSplitBK bf16 along k, 64 bytes a row.  The 16-byte groups of a
// row (8 values of k, one lane's operand of one MFMA) are permuted by the
// row, so that the eight rows one LDS cycle of a 16-byte read covers, and the
// stores below, spread over all banks.
constexpr int kSplitBK = 32;
__device__ __forceinline__ int split_swz(int r) { return ((r >> 1) ^ (r >> 3)) & 3; }
// byte offset of the 8-byte group q (k = 4 q .. 4 q + 3) of row r in a plane
__device__ __forceinline__ int split_at(int r, int q) { return r * 64 + (((q >> 1) ^ split_swz(r)) << 4) + ((q & 1) << 3); }

// descriptor of an operand of `count` elements from p (below 2^32 bytes: a
// matrix holds fewer than 2^30 elements)
template <class T>
__device__ __forceinline__ BufRsrc split_rsrc(const T* p, int64_t count) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), (short)0, (int)(uint32_t)(count * (int64_t)sizeof(T)),
                                           0x00020000);
}
// whether the elements of a row of the operand at p may be loaded by dwords: a
// buffer load of dwords takes any dword address, but drops the low two bits of
// a bf16 element at an odd index
template <class ST>
__device__ __forceinline__ bool split_dwords(const ST* p, const ST* p2, int64_t ld) {
  if constexpr (sizeof(ST) == 4) return true;
  else return ((reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(p2) | (uintptr_t)(2 * ld)) & 3) == 0;
}
// W consecutive elements (W 2 or 4) at byte offset off; elements past the
// array read 0.  DWORDS: see split_dwords
template <class ST, int W>
struct SplitRaw {
  static constexpr int DW = W * (int)sizeof(ST) / 4;   // dwords
  uint32_t v[DW];
  template <bool DWORDS = true>
  __device__ __forceinline__ void load(BufRsrc r, uint32_t off) {
    if constexpr (!DWORDS && sizeof(ST) == 2) {
#pragma unroll
      for (int i = 0; i < DW; ++i) {
        const uint32_t lo = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(off + 4 * i), 0, 0);
        const uint32_t hi = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(off + 4 * i + 2), 0, 0);
        v[i] = lo | (hi << 16);
      }
    } else if constexpr (DW == 4) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
      v[0] = x[0]; v[1] = x[1]; v[2] = x[2]; v[3] = x[3];
    } else if constexpr (DW == 2) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
      v[0] = x[0]; v[1] = x[1];
    } else {
      v[0] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
    }
  }
  __device__ __forceinline__ float at(int i) const {
    if constexpr (sizeof(ST) == 4) return __uint_as_float(v[i]);
    else return (i & 1) ? __uint_as_float(v[i >> 1] & 0xFFFF0000u) : __uint_as_float(v[i >> 1] << 16);
  }
};

// Loaders.  fetch(k0) issues a slice's global loads (unconditionally, at
// offsets clamped into the operand, so that they are one run of loads); put()
// splits the values and stores them.  Rows past the operand's end hold other
// rows' values: they only reach outputs outside the matrix, which nobody
// writes.  Terms past the contraction's end are zeroed.

// element (r, k) at base[row(r) ld + k] (+ base2[...] when FUSED): contiguous
// along k; row(r) = rows[r] when GATHER
template <int R, bool FUSED, bool GATHER, class ST = float>
struct SplitK {
  static constexpr int NV = R * 8 / kThreads;
  static_assert(NV >= 1 && R * 8 % kThreads == 0, "whole items per thread");
  BufRsrc rs, rs2;
  int K, kend;
  bool dwords;
  uint32_t off[NV];
  SplitRaw<ST, 4> a[NV], b[FUSED ? NV : 1];
  // count: elements of the operand's array from base
  __device__ SplitK(const ST* base, const ST* base2, int64_t count, int64_t ld, int row0, int nrows, int K_,
                    const int* rows = nullptr)
      : K(K_), kend(0) {
    rs = split_rsrc(base, count);
    rs2 = FUSED ? split_rsrc(base2, count) : rs;
    dwords = split_dwords(base, FUSED ? base2 : base, ld);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int idx = threadIdx.x + kThreads * i;
      int row = row0 + (idx >> 3);
      row = row < nrows ? row : nrows - 1;
      if (GATHER) row = rows[row];
      off[i] = (uint32_t)((int64_t)row * ld + 4 * (idx & 7)) * (uint32_t)sizeof(ST);
    }
  }
  template <bool DWORDS>
  __device__ __forceinline__ void load(int k0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const uint32_t o = off[i] + (uint32_t)k0 * (uint32_t)sizeof(ST);
      a[i].template load<DWORDS>(rs, o);
      if constexpr (FUSED) b[i].template load<DWORDS>(rs2, o);
    }
  }
  __device__ __forceinline__ void fetch(int k0) {
    kend = K - k0;
    if (sizeof(ST) == 4 || dwords) load<true>(k0);
    else load<false>(k0);
  }
  template <SplitFmt F>
  __device__ __forceinline__ void put(char* s, float scale) const {
    constexpr int PIECES = split_pieces(F);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int idx = threadIdx.x + kThreads * i, r = idx >> 3, q = idx & 7;
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = a[i].at(e);
        if constexpr (FUSED) x[e] += b[i].at(e);
      }
      if (kend < kSplitBK) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = 4 * q + e < kend ? x[e] : 0.f;
      }
      uint32_t p0[PIECES], p1[PIECES];
      split_pair<F>(x[0], x[1], scale, p0);
      split_pair<F>(x[2], x[3], scale, p1);
      char* d = s + split_at(r, q);
#pragma unroll
      for (int p = 0; p < PIECES; ++p) *reinterpret_cast<u32x2*>(d + p * R * 64) = u32x2{p0[p], p1[p]};
    }
  }
};

// element (r, k) at base[krow(k) ld + r] (+ base2): contiguous along r;
// krow(k) = rows[k] when GATHER.  A thread takes 4 k x RW r.
template <int R, bool FUSED, bool GATHER, class ST = float>
struct SplitR {
  static constexpr int RW = R >= 128 ? 4 : 2;
  static constexpr int NV = R / RW * 8 / kThreads;
  static_assert(NV >= 1 && R / RW * 8 % kThreads == 0, "whole items per thread");
  // lanes of a wave side by side along r: 64 bytes of a row of the array
  static constexpr int RL = RW == 4 ? 4 : 8;
  BufRsrc rs, rs2;
  const int* rows;
  uint32_t ldb;
  int K, kend;
  bool dwords;
  uint32_t col[NV];
  SplitRaw<ST, RW> a[NV][4], b[FUSED ? NV : 1][4];
  static __device__ __forceinline__ int item_r(int idx) { return RW * ((idx / (8 * RL)) * RL + idx % RL); }
  static __device__ __forceinline__ int item_q(int idx) { return (idx / RL) & 7; }
  __device__ SplitR(const ST* base, const ST* base2, int64_t count, int64_t ld, int r0, int nr, int K_,
                    const int* rows_ = nullptr)
      : rows(rows_), K(K_), kend(0) {
    rs = split_rsrc(base, count);
    rs2 = FUSED ? split_rsrc(base2, count) : rs;
    dwords = split_dwords(base, FUSED ? base2 : base, ld);
    ldb = (uint32_t)(ld * (int64_t)sizeof(ST));
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int r = r0 + item_r(threadIdx.x + kThreads * i);
      col[i] = (uint32_t)(r < nr ? r : nr - 1) * (uint32_t)sizeof(ST);
    }
  }
  __device__ __forceinline__ void fetch(int k0) {
    kend = K - k0;
    int kr[NV][4];
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = k0 + 4 * item_q(threadIdx.x + kThreads * i) + j, kc = k < K ? k : K - 1;
        kr[i][j] = GATHER ? rows[kc] : kc;
      }
    if (sizeof(ST) == 4 || dwords) load<true>(kr);
    else load<false>(kr);
  }
  template <bool DWORDS>
  __device__ __forceinline__ void load(const int (&kr)[NV][4]) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t o = (uint32_t)kr[i][j] * ldb + col[i];
        a[i][j].template load<DWORDS>(rs, o);
        if constexpr (FUSED) b[i][j].template load<DWORDS>(rs2, o);
      }
  }
  template <SplitFmt F>
  __device__ __forceinline__ void put(char* s, float scale) const {
    constexpr int PIECES = split_pieces(F);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int idx = threadIdx.x + kThreads * i, r = item_r(idx), q = item_q(idx);
#pragma unroll
      for (int e = 0; e < RW; ++e) {
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          x[j] = a[i][j].at(e);
          if constexpr (FUSED) x[j] += b[i][j].at(e);
        }
        if (kend < kSplitBK) {
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] = 4 * q + j < kend ? x[j] : 0.f;
        }
        uint32_t p0[PIECES], p1[PIECES];
        split_pair<F>(x[0], x[1], scale, p0);
        split_pair<F>(x[2], x[3], scale, p1);
        char* d = s + split_at(r + e, q);
#pragma unroll
        for (int p = 0; p < PIECES; ++p) *reinterpret_cast<u32x2*>(d + p * R * 64) = u32x2{p0[p], p1[p]};
      }
    }
  }
};

// C[BM x BN] = A[BM x K] B[K x BN] (times the scales), 4 waves in a WM x WN
// grid of TM x TN MFMA blocks each; accumulators laid out as MfmaTile's.
// NBUF 2: two copies of the slices in LDS, one barrier a slice: while a slice
// feeds the MFMAs the next one, already in registers, is split and stored and
// the one after it is loaded; NBUF 1: one copy and two barriers, for tiles
// whose two copies would leave one workgroup per CU.  A second set of
// accumulators keeps the sums that are rounded short: kAccFlush adds the
// products into it and it into the result every kSplitFlush slices, kAccSplit
// keeps every product but the first pieces' in it (for contractions that the
// caller slices itself).
constexpr int kSplitFlush = 8;
enum SplitAcc { kAccOne, kAccFlush, kAccSplit };
template <int BM, int BN, int WM, int WN, SplitFmt F, SplitAcc ACC, int NBUF = 2>
struct SplitTile {
  static constexpr int PIECES = split_pieces(F);
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int TM = WTM / 32, TN = WTN / 32;
  static constexpr int SA = PIECES * BM * 64, SB = PIECES * BN * 64;
  static constexpr int LDS_BYTES = NBUF * (SA + SB);
  static constexpr bool TWO = ACC != kAccOne;
  static_assert(WM * WN == 4, "4 waves");
  static_assert(TM >= 1 && TN >= 1 && WTM % 32 == 0 && WTN % 32 == 0, "32x32 blocks");

  f32x16 acc[TM][TN];                                // the result after run()
  f32x16 part[TWO ? TM : 1][TWO ? TN : 1];
  int wm, wn, lane;

  __device__ SplitTile() {
    lane = lane_id();
    wm = wave_id() / WN;
    wn = wave_id() % WN;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc[i][j][v] = 0.f;
          if constexpr (TWO) part[i][j][v] = 0.f;
        }
  }
  // tile-relative row / column of accumulator element (tm, tn, v)
  __device__ __forceinline__ int row(int tm, int v) const { return wm * WTM + tm * 32 + mfma32_row(v, lane); }
  __device__ __forceinline__ int col(int tn) const { return wn * WTN + tn * 32 + (lane & 31); }

  __device__ __forceinline__ void compute(const char* As, const char* Bs) {
    const int kh = lane >> 5, l32 = lane & 31;
#pragma unroll
    for (int ks = 0; ks < kSplitBK / 16; ++ks) {
      u32x4 a[TM][PIECES], b[TN][PIECES];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int p = 0; p < PIECES; ++p)
          a[i][p] = *reinterpret_cast<const u32x4*>(As + p * BM * 64 + split_at(wm * WTM + i * 32 + l32, 4 * ks + 2 * kh));
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int p = 0; p < PIECES; ++p)
          b[j][p] = *reinterpret_cast<const u32x4*>(Bs + p * BN * 64 + split_at(wn * WTN + j * 32 + l32, 4 * ks + 2 * kh));
      // the small products first
#pragma unroll
      for (int s = PIECES - 1; s >= 0; --s)
#pragma unroll
        for (int p = 0; p <= s; ++p)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              f32x16& c = (ACC == kAccFlush || (ACC == kAccSplit && s > 0)) ? part[TWO ? i : 0][TWO ? j : 0] : acc[i][j];
              c = split_mfma<F>(a[i][p], b[j][s - p], c);
            }
    }
  }
  __device__ __forceinline__ void flush() {
    if constexpr (TWO) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            acc[i][j][v] += part[i][j][v];
            part[i][j][v] = 0.f;
          }
    }
  }

  // acc += A B over K terms; sa, sb: the operands' scales (kF16x2)
  template <class LA, class LB>
  __device__ void run(LA& la, LB& lb, int K, char* smem, float sa = 1.f, float sb = 1.f) {
    const int nk = (K + kSplitBK - 1) / kSplitBK;
    if (nk == 0) return;
    la.fetch(0);
    lb.fetch(0);
    la.template put<F>(smem, sa);
    lb.template put<F>(smem + SA, sb);
    if (nk > 1) {
      la.fetch(kSplitBK);
      lb.fetch(kSplitBK);
    }
    __syncthreads();
    for (int kb = 0; kb < nk; ++kb) {
      const bool more = kb + 1 < nk;
      if constexpr (NBUF == 2) {
        char* cur = smem + (kb & 1) * (SA + SB);
        char* nxt = smem + ((kb & 1) ^ 1) * (SA + SB);
        if (more) {
          la.template put<F>(nxt, sa);
          lb.template put<F>(nxt + SA, sb);
        }
        if (kb + 2 < nk) {
          la.fetch((kb + 2) * kSplitBK);
          lb.fetch((kb + 2) * kSplitBK);
        }
        compute(cur, cur + SA);
      } else {
        compute(smem, smem + SA);
        __syncthreads();
        if (more) {
          la.template put<F>(smem, sa);
          lb.template put<F>(smem + SA, sb);
        }
        if (kb + 2 < nk) {
          la.fetch((kb + 2) * kSplitBK);
          lb.fetch((kb + 2) * kSplitBK);
        }
      }
      if (ACC == kAccFlush && kb % kSplitFlush == kSplitFlush - 1) flush();
      __syncthreads();
    }
    flush();
  }
};

}  // namespace glr
