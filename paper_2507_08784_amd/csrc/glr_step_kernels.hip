// Per-step kernels of the GreedyLore compression path on gfx950:
//   worker mean with error feedback, Approx-Top-r scores (MFMA GEMM with a
//   fused Philox/Box-Muller epilogue), top-r selection, projection,
//   fused residual + worker mean + reconstruction + optimizer.
#include "glr_device.hpp"
#include "glr_internal.hpp"
#include "glr_split.hpp"

#include <type_traits>

namespace glr {

// ---------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------
__global__ void k_fill_zero(uint32_t* p, size_t nwords) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < nwords; i += stride) p[i] = 0u;
}

__global__ void k_eye(float* Ut, int64_t d) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < d * d; i += stride) Ut[i] = (i / d == i % d) ? 1.0f : 0.0f;
}

static inline int grid_for(int64_t n, int per_thread = 1) {
  int64_t g = (n + (int64_t)kThreads * per_thread - 1) / ((int64_t)kThreads * per_thread);
  if (g < 1) g = 1;
  if (g > 2048 * 8) g = 2048 * 8;
  return (int)g;
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  size_t words = bytes / 4;
  if (!words) return hipSuccess;
  hipLaunchKernelGGL(k_fill_zero, dim3(grid_for((int64_t)words, 4)), dim3(kThreads), 0, s,
                     (uint32_t*)p, words);
  return hipGetLastError();
}

__global__ void k_absmax(const float* __restrict__ p, int64_t n, float* __restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  float mx = 0.f;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride) mx = fmaxf(mx, fabsf(p[i]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  // (bits of non-negative floats order as unsigned integers)
  if (lane_id() == 0 && mx > 0.f) atomicMax((unsigned int*)out, __float_as_uint(mx));
}
hipError_t launch_absmax(const float* p, int64_t n, float* out, hipStream_t s) {
  hipError_t e = launch_fill_zero(out, 4, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_absmax, dim3(grid_for(n, 16)), dim3(kThreads), 0, s, p, n, out);
  return hipGetLastError();
}

hipError_t launch_eye(float* Ut, int64_t d, hipStream_t s) {
  hipLaunchKernelGGL(k_eye, dim3(grid_for(d * d, 4)), dim3(kThreads), 0, s, Ut, d);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// S1 + S2: Mbar = Ebar + (1/N) sum_i G^(i)   (m x n layout; Ebar is the mean
// of the workers' error buffers left by the previous step; G in the storage
// type ST)
// ---------------------------------------------------------------------------
template <class ST>
__device__ __forceinline__ void ef_mean_at(const ST* __restrict__ G, const float* __restrict__ Ebar,
                                           float* __restrict__ Mbar, int64_t mn, int N, uint32_t* status, int check,
                                           float* __restrict__ amax, int64_t bx, int64_t gx) {
  const int64_t stride = (int64_t)gx * blockDim.x;
  bool bad = false;
  float mx = 0.f;   // the largest |Mbar| (fmaxf drops a NaN: Mbar itself still carries it)
  if ((mn & 3) == 0) {
    const int64_t q = mn >> 2;
    for (int64_t i = bx * (int64_t)blockDim.x + threadIdx.x; i < q; i += stride) {
      float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int w = 0; w < N; ++w) {
        float4 g = ld_nt_e4(G, (int64_t)w * mn + 4 * i);
        if (check) bad |= !(isfinite(g.x) && isfinite(g.y) && isfinite(g.z) && isfinite(g.w));
        acc.x += g.x; acc.y += g.y; acc.z += g.z; acc.w += g.w;
      }
      float4 e = reinterpret_cast<const float4*>(Ebar)[i];
      float4 o;
      o.x = e.x + acc.x / (float)N;
      o.y = e.y + acc.y / (float)N;
      o.z = e.z + acc.z / (float)N;
      o.w = e.w + acc.w / (float)N;
      mx = fmaxf(fmaxf(fmaxf(mx, fabsf(o.x)), fmaxf(fabsf(o.y), fabsf(o.z))), fabsf(o.w));
      reinterpret_cast<float4*>(Mbar)[i] = o;
    }
  } else {
    for (int64_t i = bx * (int64_t)blockDim.x + threadIdx.x; i < mn; i += stride) {
      float acc = 0.f;
      for (int w = 0; w < N; ++w) {
        float g = ld_e(G, (int64_t)w * mn + i);
        if (check) bad |= !isfinite(g);
        acc += g;
      }
      const float o = Ebar[i] + acc / (float)N;
      mx = fmaxf(mx, fabsf(o));
      Mbar[i] = o;
    }
  }
  if (check && bad) atomicOr(status, 1u);
  __shared__ float red[kThreads / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (lane_id() == 0) red[wave_id()] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kThreads / 64; ++w) mx = fmaxf(mx, red[w]);
    amax[bx] = mx;
  }
}
template <class ST>
__global__ void k_ef_mean(const ST* __restrict__ G, const float* __restrict__ Ebar,
                          float* __restrict__ Mbar, int64_t mn, int N, uint32_t* status,
                          int check, float* __restrict__ amax) {
  ef_mean_at(G, Ebar, Mbar, mn, N, status, check, amax, blockIdx.x, gridDim.x);
}

hipError_t launch_ef_mean(const MatView& v, bool check_finite, hipStream_t s) {
  const int64_t mn = v.m * v.n;
  if (v.st16)
    hipLaunchKernelGGL(k_ef_mean<bf16_t>, dim3(ef_mean_blocks(mn)), dim3(kThreads), 0, s, (const bf16_t*)v.G, v.Ebar,
                       v.Mbar, mn, v.N, v.status, check_finite ? 1 : 0, v.amax);
  else
    hipLaunchKernelGGL(k_ef_mean<float>, dim3(ef_mean_blocks(mn)), dim3(kThreads), 0, s, (const float*)v.G, v.Ebar,
                       v.Mbar, mn, v.N, v.status, check_finite ? 1 : 0, v.amax);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// S3b: selection scores.  C[b][j] = sum_a Mo[a][b] Ut[j][a]  (C = Mo^T U,
// D x d), never stored: the epilogue folds each column j with v_j (approx:
// lambdabar_j = u_j^T Mbar v_j) or with itself (exact: ||u_j^T Mbar||^2) and
// writes one partial per 128-row tile: part[tile][j].  Bound by the matrix
// cores, so the product runs on the fp16 ones (kF16x2): only its size against
// the rest of the same matrix matters here, so one scale for all of Mbar
// serves, from the maxima the worker mean leaves (at most 2048 floats, 2 us of
// reading).  4096 x 4096: 1332 -> 573 us (103 -> 240 TFLOP/s of fp32 products),
// 4096 x 11008: 3430 -> 1378 us, 768 x 768: 85 -> 52 us, against the fp32 MFMA
// with 16-byte loads; the scores' error against 64 bits 8.1e-7 -> 2.3e-7.
// ---------------------------------------------------------------------------
// Tiles of 128 x 128, or of 64 x 64 when the launch has fewer than kSelFew of
// the large ones, one for each CU: below that part of the chip stays idle while
// each workgroup works through its d-long contraction and its share of the
// normals.  1011 x 2053 (136 large tiles): 49 us large, 38 small; 256 x 128
// (2): 16.5 and 7.9; but the five left-sided matrices of an encoder layer (288)
// ran 3 % faster in large tiles.  Both fold 32 rows at a time in one order, so
// the scores do not depend on the choice.
constexpr int kSelFew = 256;

template <int BT, bool RIGHT, bool APPROX, bool BF16>
__device__ __forceinline__ void sel_scores_at(const float* __restrict__ Mbar, const float* __restrict__ Ut, int64_t d,
                                              int64_t D, float* __restrict__ part, uint32_t mat, uint32_t tstep,
                                              uint32_t key0, uint32_t key1, const float* __restrict__ amax,
                                              const float* __restrict__ umax, int bx, int by) {
  using T = SplitTile<BT, BT, 2, 2, BF16 ? kBf16 : kF16x2, BF16 ? kAccOne : kAccFlush>;
  __shared__ __align__(16) char smem[T::LDS_BYTES];
  __shared__ float red[2][BT];
  const int m0 = by * BT;   // rows: b in [0, D)
  const int n0 = bx * BT;   // cols: j in [0, d)
  const int em = BF16 ? 0 : split_block_exp({amax, ef_mean_blocks(d * D), 1.f, 0}, red[0]);
  const int eu = BF16 ? 0 : split_basis_exp(*umax);
  const float sm = ldexpf(1.f, em), su = ldexpf(1.f, eu);
  T tile;
  SplitK<BT, false, false> lb(Ut, nullptr, d * d, d, n0, (int)d, (int)d);
  if (RIGHT) {
    // Mo[a][b] = Mbar[b][a] : A[b][a] contiguous along a
    SplitK<BT, false, false> la(Mbar, nullptr, d * D, d, m0, (int)D, (int)d);
    tile.run(la, lb, (int)d, smem, sm, su);
  } else {
    // Mo[a][b] = Mbar[a][b] : A[b][a] contiguous along b
    SplitR<BT, false, false> la(Mbar, nullptr, d * D, D, m0, (int)D, (int)d);
    tile.run(la, lb, (int)d, smem, sm, su);
  }
  const int lane = lane_id();
  const float unscale = ldexpf(1.f, -em - eu);
#pragma unroll
  for (int tn = 0; tn < T::TN; ++tn) {
    const int j = n0 + tile.col(tn);
    float total = 0.f;
#pragma unroll
    for (int tm = 0; tm < T::TM; ++tm) {
      float acc = 0.f;   // 32 rows of column j
      if (j < d) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int b0 = m0 + tile.row(tm, 4 * g);   // multiple of 4
          if (b0 >= D) continue;
          if (APPROX) {
            float z[4];
            normals4((uint32_t)(b0 >> 2), (uint32_t)j, mat, tstep, key0, key1, z);
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (b0 + e < D) acc += tile.acc[tm][tn][4 * g + e] * unscale * z[e];
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float c = tile.acc[tm][tn][4 * g + e] * unscale;
              if (b0 + e < D) acc += c * c;
            }
          }
        }
      }
      acc += __shfl_xor(acc, 32, 64);
      total = tm == 0 ? acc : total + acc;
    }
    if (lane < 32) red[tile.wm][tile.wn * T::WTN + tn * 32 + lane] = total;
  }
  __syncthreads();
  // one partial for 64 rows: the two waves' of a small tile, each wave's of a large one
  if (threadIdx.x < BT) {
    const int j = n0 + threadIdx.x;
    if (j < d) {
      if (BT == 64) {
        part[(int64_t)by * d + j] = red[0][threadIdx.x] + red[1][threadIdx.x];
      } else {
        part[(int64_t)(2 * by) * d + j] = red[0][threadIdx.x];
        if (m0 + 64 < D) part[(int64_t)(2 * by + 1) * d + j] = red[1][threadIdx.x];
      }
    }
  }
}
template <int BT, bool RIGHT, bool APPROX, bool BF16>
__global__ void __launch_bounds__(256, BT == 64 ? 4 : 2)
k_sel_scores(const float* __restrict__ Mbar, const float* __restrict__ Ut, int64_t d, int64_t D,
             float* __restrict__ part, uint32_t mat, uint32_t tstep, uint32_t key0, uint32_t key1,
             const float* __restrict__ amax, const float* __restrict__ umax) {
  sel_scores_at<BT, RIGHT, APPROX, BF16>(Mbar, Ut, d, D, part, mat, tstep, key0, key1, amax, umax, blockIdx.x,
                                         blockIdx.y);
}

static int sel_tiles(int64_t d, int64_t D, int bt) { return (int)(((d + bt - 1) / bt) * ((D + bt - 1) / bt)); }
hipError_t launch_sel_scores(const MatView& v, bool approx, bool bf16, uint64_t seed, int64_t t, hipStream_t s) {
  if (bf16 && !approx) return hipErrorInvalidValue;
  const bool few = sel_tiles(v.d, v.D, 128) < kSelFew;
  const int bt = few ? 64 : 128;
  dim3 grid((unsigned)((v.d + bt - 1) / bt), (unsigned)((v.D + bt - 1) / bt));
  const uint32_t k0 = (uint32_t)(seed & 0xFFFFFFFFu), k1 = (uint32_t)(seed >> 32);
  const uint32_t tt = (uint32_t)((uint64_t)t & 0xFFFFFFFFu);
#define GLR_SEL1(T, R, A, B)                                                                         \
  hipLaunchKernelGGL((k_sel_scores<T, R, A, B>), grid, dim3(kThreads), 0, s, v.Mbar, v.Ut, v.d, v.D, \
                     v.lam_part, (uint32_t)v.mat, tt, k0, k1, v.amax, v.umax)
#define GLR_SEL(R, A, B)                    \
  do {                                      \
    if (few) GLR_SEL1(64, R, A, B);         \
    else GLR_SEL1(128, R, A, B);            \
  } while (0)
  if (v.right) {
    if (bf16) GLR_SEL(true, true, true);
    else if (approx) GLR_SEL(true, true, false);
    else GLR_SEL(true, false, false);
  } else {
    if (bf16) GLR_SEL(false, true, true);
    else if (approx) GLR_SEL(false, true, false);
    else GLR_SEL(false, false, false);
  }
#undef GLR_SEL
#undef GLR_SEL1
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scores and argtop_r: the tile partials of each column folded in order, then
// the r largest (descending score, ties to the smaller index; J ascending) by
// one workgroup of 1024.  It looks for the r-th largest of the
// order-preserving 32-bit keys by three passes over a histogram in LDS (11, 11
// and 10 bits; the keys, at most eight a thread, stay in registers), then
// places the winners by counting.  Bound by latency: 60 us before (a bitonic
// sort in LDS) + 9 (the fold) at d = 4096, 20 + 4 now; 8.5 + 4.3 before,
// 7.6 now at d = 128.  The selecting workgroup folds the
// partials itself up to kToprFold of them (128 KB: what one CU reads in about
// the time a launch takes); more are folded by a launch over the chip.  (Fold
// and selection in one launch, the workgroup that ends last selecting: its
// device-wide fence writes the dirty lines of the L2 back, 31 us at 4096.)
// ---------------------------------------------------------------------------
constexpr int kToprThreads = 1024;
constexpr int64_t kToprFold = 32768;
constexpr int kToprBins = 2048;
struct ToprLds {
  uint32_t hist[kToprBins];
  uint32_t wave[kToprThreads / 64];
  uint32_t pick[2];                                 // the bin found, keys above it
  uint32_t slab[8][kToprThreads / 64];
};
// the folded score of column j, in fp64: an fp32 sum of the D / 64 partials
// (squares, all positive, in the exact scores) was further off than their own
// rounding (768 x 3072: 9.5e-8 from 64 bits, 2.3e-8 so; D / 128 partials in
// fp32 7.0e-8)
__device__ __forceinline__ float fold_score(const float* __restrict__ part, int ntiles, int d, int approx, int j) {
  // 32 loads in flight: the partials come from the other XCDs' L2
  constexpr int B = 32;
  double s = 0.0;
  for (int t0 = 0; t0 < ntiles; t0 += B) {
    float x[B];
#pragma unroll
    for (int i = 0; i < B; ++i) x[i] = part[(int64_t)(t0 + i < ntiles ? t0 + i : t0) * d + j];
#pragma unroll
    for (int i = 0; i < B; ++i)
      if (t0 + i < ntiles) s += (double)x[i];
  }
  return (float)(approx ? s * s : s);
}
// folds `part` into `score` when `own`, else reads it
__device__ __forceinline__ void topr_at(const float* __restrict__ part, int ntiles, bool own, int approx, int d,
                                        float* __restrict__ score, int r, int* __restrict__ J) {
  __shared__ ToprLds L;
  constexpr int MAXQ = 8;                           // d <= 8192
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  uint32_t key[MAXQ];
  const int nq = (d + kToprThreads - 1) / kToprThreads;
#pragma unroll
  for (int q = 0; q < MAXQ; ++q) {
    const int i = tid + q * kToprThreads;
    key[q] = 0u;
    if (i < d) {
      float s;
      if (own) {
        s = fold_score(part, ntiles, d, approx, i);
        score[i] = s;
      } else {
        s = score[i];
      }
      key[q] = float_order(s);
    }
  }
  uint32_t prefix = 0, want = (uint32_t)r;          // the r-th largest has these upper bits; `want`-th among them
  int shift = 32;
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int bits = pass < 2 ? 11 : 10;
    const uint32_t mask = pass == 0 ? 0u : ~0u << shift;
    shift -= bits;
    L.hist[tid] = 0;
    L.hist[tid + kToprThreads] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MAXQ; ++q)
      if (tid + q * kToprThreads < d && (key[q] & mask) == prefix)
        atomicAdd(&L.hist[(key[q] >> shift) & ((1u << bits) - 1u)], 1u);
    __syncthreads();
    // thread t holds bins b = 2047 - 2 t and b - 1: an inclusive scan from the top
    const uint32_t h0 = L.hist[kToprBins - 1 - 2 * tid], h1 = L.hist[kToprBins - 2 - 2 * tid];
    uint32_t sum = h0 + h1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t x = __shfl_up(sum, o, 64);
      if (lane >= o) sum += x;
    }
    if (lane == 63) L.wave[w] = sum;
    __syncthreads();
    uint32_t before = 0;
    for (int i = 0; i < w; ++i) before += L.wave[i];
    const uint32_t upto = before + sum, above = upto - h0 - h1;
    if (above < want && want <= upto) {
      const bool first = want <= above + h0;
      L.pick[0] = (uint32_t)(first ? kToprBins - 1 - 2 * tid : kToprBins - 2 - 2 * tid);
      L.pick[1] = first ? above : above + h0;
    }
    __syncthreads();
    prefix |= L.pick[0] << shift;
    want -= L.pick[1];
    __syncthreads();
  }
  // every key above `prefix` and the first `want` equal to it, by index
  uint64_t gt[MAXQ], eq[MAXQ];
#pragma unroll
  for (int q = 0; q < MAXQ; ++q) {
    const bool in = tid + q * kToprThreads < d;
    gt[q] = __ballot(in && key[q] > prefix);
    eq[q] = __ballot(in && key[q] == prefix);
    if (lane == 0 && q < nq) L.slab[q][w] = (uint32_t)__popcll(gt[q]) | ((uint32_t)__popcll(eq[q]) << 16);
  }
  __syncthreads();
  uint32_t ngt = 0, neq = 0;                        // before this wave's first key, in index order
  for (int q = 0; q < nq; ++q) {
    for (int i = 0; i < kToprThreads / 64; ++i) {
      if (i == w) {
        const uint64_t lower = (1ull << lane) - 1ull;
        uint64_t g = 0, e = 0;
        uint32_t k = 0;
#pragma unroll
        for (int c = 0; c < MAXQ; ++c)
          if (c == q) { g = gt[c]; e = eq[c]; k = key[c]; }
        const uint32_t mg = ngt + (uint32_t)__popcll(g & lower), me = neq + (uint32_t)__popcll(e & lower);
        const int idx = tid + q * kToprThreads;
        if (idx < d && (k > prefix || (k == prefix && me < want))) J[mg + (me < want ? me : want)] = idx;
      }
      const uint32_t s = L.slab[q][i];
      ngt += s & 0xFFFFu;
      neq += s >> 16;
    }
  }
}
__global__ void __launch_bounds__(kToprThreads)
k_topr(const float* __restrict__ part, int ntiles, int own, int approx, int d, float* __restrict__ score, int r,
       int* __restrict__ J) {
  topr_at(part, ntiles, own != 0, approx, d, score, r, J);
}
__global__ void k_fold_scores(const float* __restrict__ part, int ntiles, int approx, int d, float* __restrict__ score) {
  const int j = blockIdx.x * (int)blockDim.x + threadIdx.x;
  if (j < d) score[j] = fold_score(part, ntiles, d, approx, j);
}

__global__ void k_iota(int* J, int r) {
  for (int i = threadIdx.x; i < r; i += blockDim.x) J[i] = i;
}

hipError_t launch_topr(const MatView& v, bool approx, hipStream_t s) {
  const int ntiles = (int)((v.D + 63) / 64);
  const bool own = v.d * ntiles <= kToprFold;
  if (!own)
    hipLaunchKernelGGL(k_fold_scores, dim3((unsigned)((v.d + 63) / 64)), dim3(64), 0, s, v.lam_part, ntiles,
                       approx ? 1 : 0, (int)v.d, v.score);
  hipLaunchKernelGGL(k_topr, dim3(1), dim3(kToprThreads), 0, s, v.lam_part, ntiles, own ? 1 : 0, approx ? 1 : 0,
                     (int)v.d, v.score, v.r, v.J);
  return hipGetLastError();
}

hipError_t launch_iota_J(const MatView& v, hipStream_t s) {
  hipLaunchKernelGGL(k_iota, dim3(1), dim3(256), 0, s, v.J, v.r);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// S4: Q^(i) = P^T M^(i), r x D per worker (both orientations), with
// P^T[k][a] = Ut[J[k]][a] and M^(i) = G^(i) + E^(i) fused into the load (G
// and E in the storage type ST, widened to fp32 as they load).  VEC: every
// operand slice loads as whole float4s (proj_vec on the host).
// ---------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN, bool RIGHT, class ST, bool VEC = false>
__device__ __forceinline__ void proj_at(const ST* __restrict__ G, const ST* __restrict__ E,
                                        const float* __restrict__ Ut, const int* __restrict__ J,
                                        float* __restrict__ Qpart, int64_t d, int64_t D, int r, int N, int kslice,
                                        int bx, int by, int bz) {
  using T = MfmaTile<BM, BN, WM, WN>;
  __shared__ __align__(16) float smem[T::LDS_FLOATS];
  const int n0 = bx * BN;   // b
  const int m0 = by * BM;   // k (rank index)
  const int w = bz % N;     // worker
  const int z = bz / N;     // slice of the d contraction
  const int64_t k0 = (int64_t)z * kslice;
  const int klen = (int)(d - k0 < kslice ? d - k0 : kslice);
  const int64_t dD = d * D;
  const ST* Gi = G + (int64_t)w * dD;
  const ST* Ei = E + (int64_t)w * dD;
  T tile;
  // fp32 accumulators are added into fp64 ones every 512 terms of the slice
  double dacc[T::TM][T::TN][16];
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) dacc[tm][tn][v] = 0.0;
  LoadK<BM, 32, false, true, float, VEC> la(Ut + k0, nullptr, d, m0, r, klen, J);
  if (RIGHT) {
    // M^(i) oriented: Mo[a][b] = M[b][a], M is D x d row-major
    LoadK<BN, 32, true, false, ST, VEC> lb(Gi + k0, Ei + k0, d, n0, (int)D, klen, nullptr);
    tile.run(la, lb, klen, smem, dacc);
  } else {
    LoadR<BN, 32, true, false, ST, VEC> lb(Gi + k0 * D, Ei + k0 * D, D, n0, (int)D, klen);
    tile.run(la, lb, klen, smem, dacc);
  }
  float* Qz = Qpart + ((int64_t)z * N + w) * r * D;
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn) {
      const int b = n0 + tile.col(tn);
      if (b >= D) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int k = m0 + tile.row(tm, v);
        if (k < r) Qz[(int64_t)k * D + b] = (float)dacc[tm][tn][v];
      }
    }
}
template <int BM, int BN, int WM, int WN, bool RIGHT, class ST, bool VEC>
__global__ void __launch_bounds__(256)
k_proj(const ST* __restrict__ G, const ST* __restrict__ E, const float* __restrict__ Ut,
       const int* __restrict__ J, float* __restrict__ Qpart, int64_t d, int64_t D, int r, int N, int kslice) {
  proj_at<BM, BN, WM, WN, RIGHT, ST, VEC>(G, E, Ut, J, Qpart, d, D, r, N, kslice, blockIdx.x, blockIdx.y, blockIdx.z);
}
// Above rank 64 the projection is bound by the matrix cores: the same product
// on the bf16 ones (kBf16x3: M^(i) has no scale known in advance, and Q's
// columns are held to their own size), the 1024-term slices of d added in fp64
// by the launch that packs Q.  11008 x 4096, r = 128: 1000 -> 757 us (122
// TFLOP/s of fp32 products), the same with bf16 storage 1030 -> 756 us,
// 8192 x 28672, r = 256, N = 4: 5.2 -> 3.7 ms, against the fp32 MFMA.
template <int BM, int WM, int WN, bool RIGHT, class ST>
struct ProjSplit {
  static constexpr int BN = 64;
  using T = SplitTile<BM, BN, WM, WN, kBf16x3, kAccSplit, BM == 256 ? 1 : 2>;
};
template <int BM, int WM, int WN, bool RIGHT, class ST>
__device__ __forceinline__ void proj_split_at(const ST* __restrict__ G, const ST* __restrict__ E,
                                              const float* __restrict__ Ut, const int* __restrict__ J,
                                              float* __restrict__ Qpart, int64_t d, int64_t D, int r, int N, int kslice,
                                              int bx, int by, int bz) {
  using PS = ProjSplit<BM, WM, WN, RIGHT, ST>;
  using T = typename PS::T;
  constexpr int BN = PS::BN;
  __shared__ __align__(16) char smem[T::LDS_BYTES];
  const int n0 = bx * BN, m0 = by * BM;   // b, rank index
  const int w = bz % N, z = bz / N;       // worker, slice of the d contraction
  const int64_t k0 = (int64_t)z * kslice, dD = d * D;
  const int klen = (int)(d - k0 < kslice ? d - k0 : kslice);
  const ST* Gi = G + (int64_t)w * dD;
  const ST* Ei = E + (int64_t)w * dD;
  T tile;
  SplitK<BM, false, true> la(Ut + k0, nullptr, d * d - k0, d, m0, r, klen, J);
  if (RIGHT) {
    // M^(i) oriented: Mo[a][b] = M[b][a], M is D x d row-major
    SplitK<BN, true, false, ST> lb(Gi + k0, Ei + k0, dD - k0, d, n0, (int)D, klen);
    tile.run(la, lb, klen, smem);
  } else {
    SplitR<BN, true, false, ST> lb(Gi + k0 * D, Ei + k0 * D, dD - k0 * D, D, n0, (int)D, klen);
    tile.run(la, lb, klen, smem);
  }
  float* Qz = Qpart + ((int64_t)z * N + w) * r * D;
#pragma unroll
  for (int tm = 0; tm < T::TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn) {
      const int b = n0 + tile.col(tn);
      if (b >= D) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int k = m0 + tile.row(tm, v);
        if (k < r) Qz[(int64_t)k * D + b] = tile.acc[tm][tn][v];
      }
    }
}
// A 1-D grid in which the gy rank tiles of a (column tile, worker, slice)
// triple are 8 blocks apart, so they run on the same XCD at the same time and
// the second read of those columns hits that XCD's L2 (blocks go to the XCDs
// in turn).
template <int BM, int WM, int WN, bool RIGHT, class ST>
__global__ void __launch_bounds__(256, 2)
k_proj_split(const ST* __restrict__ G, const ST* __restrict__ E, const float* __restrict__ Ut,
             const int* __restrict__ J, float* __restrict__ Qpart, int64_t d, int64_t D, int r, int N, int kslice,
             int gx, int gy, int ntiles) {
  const int L = blockIdx.x, xcd = L & 7, slot = L >> 3;
  const int by = slot % gy, tile = (slot / gy) * 8 + xcd;
  if (tile >= ntiles) return;
  proj_split_at<BM, WM, WN, RIGHT, ST>(G, E, Ut, J, Qpart, d, D, r, N, kslice, tile % gx, by, tile / gx);
}
// the conditions under which every loader of the projection takes its
// float4 path: rows of U^T, G and E in whole float4s (d and D multiples of
// 4, so every slice start and length is one), and the arrays aligned
static bool proj_vec(const MatView& v, size_t esz) {
  const uintptr_t al = 4 * esz - 1;
  return v.d % 4 == 0 && v.D % 4 == 0 && (reinterpret_cast<uintptr_t>(v.Ut) & 15) == 0 &&
         (reinterpret_cast<uintptr_t>(v.G) & al) == 0 && (reinterpret_cast<uintptr_t>(v.E) & al) == 0;
}

template <class ST>
static hipError_t launch_proj_st(const MatView& v, hipStream_t s) {
  const int r = v.r;
  const ST* G = static_cast<const ST*>(v.G);
  const ST* E = static_cast<const ST*>(v.E);
  const int splits = proj_splits(v.d, v.D, r, v.N);
  const int64_t kslice = proj_kslice(v.d, v.D, r, v.N);
  const bool vec = proj_vec(v, sizeof(ST));
  dim3 grid;
  grid.z = (unsigned)(v.N * splits);
#define GLR_PROJ1(BM, BN, WM, WN, R, VE)                                                            \
  hipLaunchKernelGGL((k_proj<BM, BN, WM, WN, R, ST, VE>), grid, dim3(kThreads), 0, s, G, E, v.Ut,   \
                     v.J, v.Qpart, v.d, v.D, r, v.N, (int)kslice)
#define GLR_PROJ(BM, BN, WM, WN)                                                                    \
  do {                                                                                              \
    grid.x = (unsigned)((v.D + BN - 1) / BN);                                                       \
    grid.y = (unsigned)((r + BM - 1) / BM);                                                         \
    if (v.right) {                                                                                  \
      if (vec) GLR_PROJ1(BM, BN, WM, WN, true, true);                                               \
      else GLR_PROJ1(BM, BN, WM, WN, true, false);                                                  \
    } else {                                                                                        \
      if (vec) GLR_PROJ1(BM, BN, WM, WN, false, true);                                              \
      else GLR_PROJ1(BM, BN, WM, WN, false, false);                                                 \
    }                                                                                               \
  } while (0)
  // one rank tile covers all r rows, so G and E are read once.  Up to rank
  // 64 the tile adds its fp32 sums into fp64 every 512 terms; above, the
  // slices are 1024 terms and the reduction adds them in fp64, which keeps
  // fp64 accumulators out of the larger tiles (a 128-row tile holding them
  // spills).  At rank 64 the 64 x 128 tile without the fp64 sums was 10 %
  // slower than the 64 x 64 one with them (fewer, longer blocks).
  if (r <= 32) GLR_PROJ(32, 128, 1, 4);
  else if (r <= kProjFlushRank) GLR_PROJ(64, 64, 2, 2);
#define GLR_PROJS1(BM, WM, WN, R)                                                                          \
  hipLaunchKernelGGL((k_proj_split<BM, WM, WN, R, ST>), gr, dim3(kThreads), 0, s, G, E, v.Ut, v.J, v.Qpart, \
                     v.d, v.D, r, v.N, (int)kslice, gx, gy, ntiles)
#define GLR_PROJS(BM, WM, WN)                                         \
  do {                                                                \
    const int gx = (int)((v.D + 63) / 64), gy = (r + BM - 1) / BM;    \
    const int ntiles = gx * (int)grid.z;                              \
    const dim3 gr((unsigned)(((ntiles + 7) / 8) * 8 * gy));           \
    if (v.right) GLR_PROJS1(BM, WM, WN, true);                        \
    else GLR_PROJS1(BM, WM, WN, false);                               \
  } while (0)
  else if (r <= kProjWideRank) GLR_PROJS(128, 2, 2);
  else GLR_PROJS(256, 4, 1);
#undef GLR_PROJS
#undef GLR_PROJS1
#undef GLR_PROJ
#undef GLR_PROJ1
  return hipGetLastError();
}
hipError_t launch_proj(const MatView& v, hipStream_t s) {
  return v.st16 ? launch_proj_st<bf16_t>(v, s) : launch_proj_st<float>(v, s);
}

// S6 (with the slices of the projection): Q^(i) = sum over slices of the
// partial products, Rbar = (1/N) sum_i Q^(i); both sums in a fixed order, fp64
// (Q null: the one slice is Q^(i) already)
__device__ __forceinline__ void proj_reduce_at(const float* __restrict__ part, int splits, int N, int64_t rD,
                                               float* __restrict__ Q, float* __restrict__ Rbar, int64_t bx,
                                               int64_t gx) {
  const int64_t stride = (int64_t)gx * blockDim.x;
  for (int64_t i = bx * (int64_t)blockDim.x + threadIdx.x; i < rD; i += stride) {
    double rsum = 0.0;
    for (int w = 0; w < N; ++w) {
      double q = 0.0;
      for (int z = 0; z < splits; ++z) q += (double)part[((int64_t)z * N + w) * rD + i];
      if (Q) Q[(int64_t)w * rD + i] = (float)q;
      rsum += q;
    }
    Rbar[i] = (float)(rsum / (double)N);
  }
}
__global__ void k_proj_reduce(const float* __restrict__ part, int splits, int N, int64_t rD, float* __restrict__ Q,
                              float* __restrict__ Rbar) {
  proj_reduce_at(part, splits, N, rD, Q, Rbar, blockIdx.x, gridDim.x);
}

// The same for the split residual pass (resid_packed): Q^(i) and P leave as
// fp16 pieces in the order in which its MFMAs read them, so that it needs
// neither LDS nor conversions.  A fragment is 64 lanes x 8 values of k: lane l
// holds row 32 blk + l % 32 of the operand (a column b of Q, a row a of P) at
// k = 16 ks + 8 (l / 32) ..+7; the fragment of piece p, step ks, block blk is
// at ((blk KS + ks) 2 + p) 64 (u32x4), KS the steps r is padded to with zeros.
// Each column of Q^(i), and each row of P that needs it (pack_p), has a scale of
// its own (exponents in Qe and Pe): the residual is compared and Adam normalises element by element, so
// a column or row far smaller than the rest keeps its relative precision (with
// one scale for P, rows 1e-4 of the rest were 4.6e-5 off, 1e-6 4.7e-3).
// Bound by reading the projection's slices, and for small ranks by latency.
// Up to rank 128 a wave holds all of a column (8 KS values a lane) and takes
// the 32 columns of one worker's block by itself, and other workgroups of the
// launch form Rbar from a second read of the slices (pack_waves).  Above, a
// workgroup of 1024 reads the slices of 32 columns once for all workers, in
// turn, for both (pack_block): there the second read would cost more (0.94 GB
// at 8192 x 28672), and the chain of barriers less: per launch 350 us against
// 65 of pack_waves for the fifty layers at rank 8, 143 against 96 at
// 11008 x 4096, rank 128.
constexpr int kPackThreads = 1024;
constexpr int kPackWaveSteps = 8;   // largest KS of pack_waves
constexpr SplitFmt pack_fmt(int KS) { return KS == 1 ? kBf16x3 : kF16x2; }
// one lane's part of every piece of a fragment
template <SplitFmt F>
__device__ __forceinline__ void pack_store(const float (&x)[8], float scale, u32x4* dst) {
  constexpr int PC = split_pieces(F);
  u32x4 f[PC];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t p[PC];
    split_pair<F>(x[2 * e], x[2 * e + 1], scale, p);
#pragma unroll
    for (int i = 0; i < PC; ++i) f[i][e] = p[i];
  }
#pragma unroll
  for (int i = 0; i < PC; ++i) dst[64 * i] = f[i];
}
// The KS fragments of block blk of P, by NW waves, KC = KS / NW steps (at least
// one) each.  Rows whose largest entry lies in [kUnitLow, kUnitHigh), nearly
// all of an orthonormal basis, are scaled by 2^kUnitExp (their pieces resolve
// 2^-24 of it); a row outside, by a power of its own: Pe holds its exponent
// beyond kUnitExp and, past the rows, whether a block has any.  The residual
// then corrects that block's products; doing so for every block cost it 12 % at
// rank 128 (registers of loads in flight).  red: 32 floats a wave.
constexpr float kUnitLow = 0x1p-7f, kUnitHigh = 0x1p+9f;
template <SplitFmt F, int NW, int KC>
__device__ __forceinline__ void pack_p(int blk, int r, int KS, int64_t d, const float* __restrict__ Ut,
                                       const int* __restrict__ J, u32x4* __restrict__ Pf, int* __restrict__ Pe,
                                       float* red) {
  const int lane = lane_id(), w = NW == 1 ? 0 : wave_id(), k0 = w * KC;
  const int a = blk * 32 + (lane & 31);
  float x[KC][8], scale = 1.f;
#pragma unroll
  for (int ks = 0; ks < KC; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 16 * (k0 + ks) + 8 * (lane >> 5) + e;
      x[ks][e] = (k < r && a < d) ? Ut[(int64_t)J[k] * d + a] : 0.f;
    }
  if constexpr (F == kF16x2) {
    float mx = 0.f;
#pragma unroll
    for (int ks = 0; ks < KC; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(x[ks][e]));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (lane < 32) red[w * 32 + lane] = mx;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NW; ++i) mx = fmaxf(mx, red[i * 32 + (lane & 31)]);
    const int own = mx >= kUnitLow && mx < kUnitHigh ? 0 : mx > 0.f ? split_exp(mx) - kUnitExp : 0;
    const uint64_t odd = __ballot(own != 0);
    if (w == 0 && lane < 32) Pe[blk * 32 + lane] = own;
    if (w == 0 && lane == 0) Pe[(int64_t)((d + 31) / 32) * 32 + blk] = odd != 0;
    scale = ldexpf(1.f, kUnitExp + own);
  }
#pragma unroll
  for (int ks = 0; ks < KC; ++ks)
    if (k0 + ks < KS)
      pack_store<F>(x[ks], scale, Pf + ((int64_t)blk * KS + k0 + ks) * (64 * split_pieces(F)) + lane);
}
// blocks of kThreads: four fragments columns of Q each, then a block of P each
// (four at one step), then Rbar
struct PackGrid {
  int q, p, rbar;
};
__host__ __device__ inline PackGrid pack_grid(int64_t d, int64_t D, int N, int r, int KS) {
  const int64_t q = (D + 31) / 32 * N, p = (d + 31) / 32, rb = ((int64_t)r * D + kThreads - 1) / kThreads;
  return {(int)((q + 3) / 4), KS == 1 ? (int)((p + 3) / 4) : (int)p, (int)rb};
}
template <int KS>
__device__ __forceinline__ void pack_waves(const float* __restrict__ part, int splits, int N, int r, int64_t d,
                                           int64_t D, const float* __restrict__ Ut, const int* __restrict__ J,
                                           u32x4* __restrict__ Qf, int* __restrict__ Qe, u32x4* __restrict__ Pf,
                                           int* __restrict__ Pe, float* __restrict__ Rbar, int bid) {
  const PackGrid g = pack_grid(d, D, N, r, KS);
  const int64_t rD = (int64_t)r * D;
  const int lane = lane_id();
  if (bid < g.q) {
    const int item = bid * 4 + wave_id(), nqb = (int)((D + 31) / 32);
    if (item >= nqb * N) return;
    const int w = item / nqb, blk = item % nqb;
    const int64_t b = (int64_t)blk * 32 + (lane & 31);
    // a run of 16 loads a slice (KC steps at a time: fp64 sums of all of them
    // would leave two waves per SIMD), the row as the scalar part of the
    // address; what lies past r is dropped below
    constexpr int KC = KS < 2 ? KS : 2;
    const uint32_t off = (uint32_t)((8 * (lane >> 5) * D + (b < D ? b : D - 1)) * 4);
    float x[KS][8], mx = 0.f;
#pragma unroll
    for (int k0 = 0; k0 < KS; k0 += KC) {
      double s[KC][8];
#pragma unroll
      for (int ks = 0; ks < KC; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) s[ks][e] = 0.0;
      for (int z = 0; z < splits; ++z) {
        const BufRsrc pz = buf_rsrc(part + ((int64_t)z * N + w) * rD, (uint32_t)(rD * 4));
        float t[KC][8];
#pragma unroll
        for (int ks = 0; ks < KC; ++ks)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int k = 16 * (k0 + ks) + e < r ? 16 * (k0 + ks) + e : 0;
            t[ks][e] =
                __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(pz, (int)off, (int)(uint32_t)(k * D * 4), 0));
          }
#pragma unroll
        for (int ks = 0; ks < KC; ++ks)
#pragma unroll
          for (int e = 0; e < 8; ++e) s[ks][e] += (double)t[ks][e];
      }
#pragma unroll
      for (int ks = 0; ks < KC; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          x[k0 + ks][e] = (16 * (k0 + ks) + 8 * (lane >> 5) + e < r && b < D) ? (float)s[ks][e] : 0.f;
          mx = fmaxf(mx, fabsf(x[k0 + ks][e]));
        }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const int e2 = split_exp(mx);
    if (lane < 32) Qe[(int64_t)item * 32 + lane] = e2;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      if (KS > 1 || r > 8 || lane < 32)
        pack_store<pack_fmt(KS)>(x[ks], ldexpf(1.f, e2),
                                 Qf + ((int64_t)item * KS + ks) * (64 * split_pieces(pack_fmt(KS))) + lane);
  } else if (bid < g.q + g.p) {
    if constexpr (KS == 1) {
      const int blk = (bid - g.q) * 4 + wave_id();
      if (blk < (int)((d + 31) / 32)) pack_p<pack_fmt(KS), 1, 1>(blk, r, KS, d, Ut, J, Pf, Pe, nullptr);
    } else {
      __shared__ float red[4 * 32];
      pack_p<pack_fmt(KS), 4, (KS + 3) / 4>(bid - g.q, r, KS, d, Ut, J, Pf, Pe, red);
    }
  } else {
    const int64_t i = (int64_t)(bid - g.q - g.p) * kThreads + threadIdx.x;
    if (i >= rD) return;
    double rsum = 0.0;
    for (int w = 0; w < N; ++w) {
      double q = 0.0;
      for (int z = 0; z < splits; ++z) q += (double)part[((int64_t)z * N + w) * rD + i];
      rsum += q;
    }
    Rbar[i] = (float)(rsum / (double)N);
  }
}
__device__ __forceinline__ void pack_block(const float* __restrict__ part, int splits, int N, int r, int KS, int64_t d,
                                        int64_t D, const float* __restrict__ Ut, const int* __restrict__ J,
                                        u32x4* __restrict__ Qf, int* __restrict__ Qe, u32x4* __restrict__ Pf,
                                        int* __restrict__ Pe, float* __restrict__ Rbar, int bid, float* dyn) {
  const int tid = threadIdx.x, nqb = (int)((D + 31) / 32);
  if (bid >= nqb) {
    static_assert(kPackRank == 16 * (kPackThreads / 64), "a wave a step");
    pack_p<kF16x2, kPackThreads / 64, 1>(bid - nqb, r, KS, d, Ut, J, Pf, Pe, dyn);
    return;
  }
  constexpr int KG = kPackThreads / 32;            // rows of k side by side
  constexpr int MAXK = kPackRank / KG;             // rows of k per thread
  float* tile = dyn;                               // 16 KS x 33
  float* red = dyn + 16 * KS * 33;                 // (waves) x 32
  const int c = tid & 31, kg = tid >> 5;
  const int64_t b = (int64_t)bid * 32 + c, rD = (int64_t)r * D;
  double rsum[MAXK];
#pragma unroll
  for (int q = 0; q < MAXK; ++q) rsum[q] = 0.0;
  for (int w = 0; w < N; ++w) {
    float mx = 0.f;
#pragma unroll
    for (int q = 0; q < MAXK; ++q) {
      const int k = kg + q * KG;
      if (k >= 16 * KS) break;
      double s = 0.0;
      if (k < r && b < D)
        for (int z = 0; z < splits; ++z) s += (double)part[((int64_t)z * N + w) * rD + (int64_t)k * D + b];
      rsum[q] += s;
      tile[k * 33 + c] = (float)s;
      mx = fmaxf(mx, fabsf((float)s));
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if ((tid & 63) < 32) red[(tid >> 6) * 32 + c] = mx;
    __syncthreads();
    mx = 0.f;
#pragma unroll
    for (int i = 0; i < kPackThreads / 64; ++i) mx = fmaxf(mx, red[i * 32 + c]);
    const int e2 = split_exp(mx);
    if (tid < 32) Qe[((int64_t)w * nqb + bid) * 32 + c] = e2;
    if (tid < KS * 64) {
      const int lane = tid & 63, ks = tid >> 6;    // lane & 31 == c
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = tile[(16 * ks + 8 * (lane >> 5) + e) * 33 + c];
      pack_store<kF16x2>(x, ldexpf(1.f, e2), Qf + (((int64_t)w * nqb + bid) * KS + ks) * 128 + lane);
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < MAXK; ++q) {
    const int k = kg + q * KG;
    if (k < r && b < D) Rbar[(int64_t)k * D + b] = (float)(rsum[q] / (double)N);
  }
}
static size_t pack_lds(int KS) { return ((size_t)16 * KS * 33 + (size_t)kPackThreads / 64 * 32) * 4; }
static int pack_blocks(int64_t d, int64_t D, int N, int r) {
  const int KS = pack_steps(r);
  if (KS <= kPackWaveSteps) {
    const PackGrid g = pack_grid(d, D, N, r, KS);
    return g.q + g.p + g.rbar;
  }
  return (int)((D + 31) / 32 + (d + 31) / 32);
}
__global__ void __launch_bounds__(kPackThreads)
k_pack_block(const float* __restrict__ part, int splits, int N, int r, int KS, int64_t d, int64_t D,
             const float* __restrict__ Ut, const int* __restrict__ J, u32x4* __restrict__ Qf, int* __restrict__ Qe,
             u32x4* __restrict__ Pf, int* __restrict__ Pe, float* __restrict__ Rbar) {
  extern __shared__ __align__(16) unsigned char dyn[];
  pack_block(part, splits, N, r, KS, d, D, Ut, J, Qf, Qe, Pf, Pe, Rbar, blockIdx.x, reinterpret_cast<float*>(dyn));
}
template <int KS>
__global__ void __launch_bounds__(kThreads)
k_pack_waves(const float* __restrict__ part, int splits, int N, int r, int64_t d, int64_t D,
             const float* __restrict__ Ut, const int* __restrict__ J, u32x4* __restrict__ Qf, int* __restrict__ Qe,
             u32x4* __restrict__ Pf, int* __restrict__ Pe, float* __restrict__ Rbar) {
  pack_waves<KS>(part, splits, N, r, d, D, Ut, J, Qf, Qe, Pf, Pe, Rbar, blockIdx.x);
}

hipError_t launch_rbar(const MatView& v, hipStream_t s) {
  const int splits = proj_splits(v.d, v.D, v.r, v.N);
  if (v.packed) {
    const int KS = pack_steps(v.r);
    const dim3 grid((unsigned)pack_blocks(v.d, v.D, v.N, v.r));
#define GLR_PW(K)                                                                                                  \
  hipLaunchKernelGGL(k_pack_waves<K>, grid, dim3(kThreads), 0, s, v.Qpart, splits, v.N, v.r, v.d, v.D, v.Ut, v.J, \
                     (u32x4*)v.Qf, v.Qe, (u32x4*)v.Pf, v.Pe, v.Rbar)
    switch (KS) {
      case 1: GLR_PW(1); break;
      case 2: GLR_PW(2); break;
      case 4: GLR_PW(4); break;
      case 8: GLR_PW(8); break;
      default:
        hipLaunchKernelGGL(k_pack_block, grid, dim3(kPackThreads), pack_lds(KS), s, v.Qpart, splits, v.N, v.r, KS, v.d,
                           v.D, v.Ut, v.J, (u32x4*)v.Qf, v.Qe, (u32x4*)v.Pf, v.Pe, v.Rbar);
    }
    static_assert(kPackWaveSteps == 8, "one variant per KS");
#undef GLR_PW
    return hipGetLastError();
  }
  const int64_t rD = (int64_t)v.r * v.D;
  hipLaunchKernelGGL(k_proj_reduce, dim3(grid_for(rD)), dim3(kThreads), 0, s, v.Qpart, splits, v.N, rD,
                     v.Qpart == v.Q ? nullptr : v.Q, v.Rbar);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// S5 + S7 + S8 fused, one pass over the m x n layout, up to rank 256:
//   C^(i) = P Q^(i) in the caller's layout
//   E^(i) <- (G^(i) - C^(i)) + E^(i)
//   Ghat  = (1/N) sum_i C^(i) (= P Rbar by linearity);
//   Ebar  = the mean of the stored E^(i) (summed in registers as they are
//   written: Mbar - Ghat equals it in real arithmetic, but when the residual
//   is small against Mbar that difference keeps only the low bits of two
//   nearly equal fp32 values);
//   optimizer on X with Ghat.
// A wave owns a 32 x 32 tile of the layout for all workers: the pieces of P
// for its rows (columns when RIGHT) stay in its registers, those of Q^(i) come
// as fragments straight from the cache (k_pack), and there is no LDS and no
// barrier, so that the waves of a CU drift apart and the loads of some cover
// the products of others.  MFMA lanes are tile columns, so that a load or
// store of one accumulator register moves whole 128-byte rows of 32 columns
// (partial-line writes make the memory side fetch the line first).  The
// product of the first pieces goes into one accumulator, the others into
// another: the sums that the large one rounds are a third as many.
// Bound by HBM: G and E in, E out, X, the optimizer state and Ebar.  Before
// (fp32 MFMA on LDS slices, P Rbar as a product of its own): 4096 x 4096,
// r = 64, N = 8: 496 -> 382 us (5.4 TB/s, the rate of a large copy);
// 11008 x 4096, r = 128: 1890 -> 1210 us; the same in bf16: 1705 -> 1072 us;
// 8192 x 28672, r = 256, N = 4: 6.73 -> 5.11 ms.
// ---------------------------------------------------------------------------
template <int OPT, bool RIGHT, int KS, class ST>
__device__ __forceinline__ void resid_packed_at(const ST* __restrict__ G, ST* __restrict__ E, float* __restrict__ Ebar,
                                                const u32x4* __restrict__ Qf, const int* __restrict__ Qe,
                                                const u32x4* __restrict__ Pf, const int* __restrict__ Pe,
                                                float* __restrict__ X,
                                                float* __restrict__ S1, float* __restrict__ S2, int64_t m, int64_t n,
                                                int r, int N, const OptParams& op, int bx, int by) {
  const int lane = lane_id(), wv = wave_id(), live = r <= 8 ? 32 : 64;
  const int64_t r0 = (int64_t)by * 64 + (wv >> 1) * 32, c0 = (int64_t)bx * 64 + (wv & 1) * 32;
  if (r0 >= m || c0 >= n) return;
  const int64_t mn = m * n;
  const int64_t nqb = ((RIGHT ? m : n) + 31) / 32, qblk = (RIGHT ? r0 : c0) / 32, pblk = (RIGHT ? c0 : r0) / 32;
  constexpr SplitFmt F = pack_fmt(KS);
  constexpr int PC = split_pieces(F);
  u32x4 pp[KS][PC];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int i = 0; i < PC; ++i) pp[ks][i] = Pf[((pblk * KS + ks) * PC + i) * 64 + lane];
  const int podd = F == kF16x2 ? __builtin_amdgcn_readfirstlane(Pe[((RIGHT ? n : m) + 31) / 32 * 32 + pblk]) : 0;
  // every m x n array is addressed as a buffer (m n 4 < 2^32 bytes): a uniform
  // descriptor and one 32-bit byte offset per element, shared by all of them;
  // elements outside the matrix take kBufNone
  const int64_t cc = c0 + (lane & 31);
  uint32_t ob[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int64_t row = r0 + mfma32_row(v, lane);
    ob[v] = (cc < n && row < m) ? (uint32_t)((row * n + cc) * 4) : kBufNone;
  }
  float esum[16], gsum[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) esum[v] = gsum[v] = 0.f;
  // (two copies of the loop: the common one keeps its registers and schedule)
  auto workers = [&](auto odd) {
    constexpr bool ODD = decltype(odd)::value;
    for (int w = 0; w < N; ++w) {
      const BufRsrc Gi = buf_rsrc_s(G + (int64_t)w * mn, mn);
      const BufRsrc Ei = buf_rsrc_s(E + (int64_t)w * mn, mn);
      float gv[16], eo[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        gv[v] = buf_lde<ST>(Gi, ob[v]);
        eo[v] = buf_lde<ST>(Ei, ob[v]);
      }
      const u32x4* q = Qf + ((int64_t)w * nqb + qblk) * (KS * PC * 64) + lane;
      const int* qe = Qe + ((int64_t)w * nqb + qblk) * 32;
      f32x16 big, small;
#pragma unroll
      for (int v = 0; v < 16; ++v) big[v] = small[v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        u32x4 qq[PC];
        if constexpr (KS == 1) {
          // rank 8 or less: the upper lanes hold zeros and load nothing
#pragma unroll
          for (int i = 0; i < PC; ++i) qq[i] = u32x4{0u, 0u, 0u, 0u};
          if (lane < live) {
#pragma unroll
            for (int i = 0; i < PC; ++i) qq[i] = q[i * 64];
          }
        } else {
#pragma unroll
          for (int i = 0; i < PC; ++i) qq[i] = q[(ks * PC + i) * 64];
        }
        // piece i of P times piece s - i of Q, the smallest products first
#pragma unroll
        for (int s = PC - 1; s >= 0; --s)
#pragma unroll
          for (int i = 0; i <= s; ++i) {
            f32x16& c = s == 0 ? big : small;
            c = RIGHT ? split_mfma<F>(qq[s - i], pp[ks][i], c) : split_mfma<F>(pp[ks][i], qq[s - i], c);
          }
      }
      if constexpr (ODD) {
        // rows of P that are packed by exponents of their own
        const int* pe = Pe + pblk * 32;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int4 x = RIGHT ? make_int4(pe[lane & 31], pe[lane & 31], pe[lane & 31], pe[lane & 31])
                               : *reinterpret_cast<const int4*>(pe + 8 * g + 4 * (lane >> 5));
          const int xe[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            big[4 * g + e] = ldexpf(big[4 * g + e], -xe[e]);
            small[4 * g + e] = ldexpf(small[4 * g + e], -xe[e]);
          }
        }
      }
      // columns of Q are tile rows (RIGHT) or this lane's column
      int ex[RIGHT ? 16 : 1];
      if (RIGHT) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int4 x = *reinterpret_cast<const int4*>(qe + 8 * g + 4 * (lane >> 5));
          ex[RIGHT ? 4 * g : 0] = x.x; ex[RIGHT ? 4 * g + 1 : 0] = x.y;
          ex[RIGHT ? 4 * g + 2 : 0] = x.z; ex[RIGHT ? 4 * g + 3 : 0] = x.w;
        }
      } else {
        ex[0] = qe[lane & 31];
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float s = big[v] + small[v];
        const float c = F == kF16x2 ? ldexpf(s, -ex[RIGHT ? v : 0] - kUnitExp) : s;
        // (G - P Q) + E: G and P Q nearly cancel, E is the small part
        const float e = (gv[v] - c) + eo[v];
        buf_ste<ST>(Ei, ob[v], e);
        esum[v] += stored<ST>(e);
        gsum[v] += c;
      }
    }
  };
  if (podd) workers(std::true_type{});
  else workers(std::false_type{});
  const uint32_t bytes = (uint32_t)(mn * 4);
  const BufRsrc Xr = buf_rsrc(X, bytes), S1r = buf_rsrc(S1, bytes), Ebr = buf_rsrc(Ebar, bytes);
  const BufRsrc S2r = buf_rsrc(OPT == 1 ? S2 : S1, bytes);
  const float inv_n = 1.0f / (float)N;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint32_t o = ob[v];
    const float gh = gsum[v] * inv_n;
    float xv = buf_ld(Xr, o);
    float s1 = buf_ld(S1r, o);
    if (OPT == 0) {
      s1 = op.beta1 * s1 + (1.0f - op.beta1) * gh;
      xv = xv - op.lr * s1;
    } else {
      float s2 = buf_ld(S2r, o);
      s1 = op.beta1 * s1 + (1.0f - op.beta1) * gh;
      s2 = op.beta2 * s2 + (1.0f - op.beta2) * gh * gh;
      xv = xv - op.lr * s1 / (sqrtf(s2) + op.eps);
      buf_st(S2r, o, s2);
    }
    buf_st(S1r, o, s1);
    buf_st(Ebr, o, esum[v] * inv_n);
    buf_st(Xr, o, xv);
  }
}
// registers: 8 KS for P, so two waves per SIMD up to rank 256
template <int OPT, bool RIGHT, int KS, class ST>
__global__ void __launch_bounds__(256, KS <= 4 ? 3 : 2)
k_resid_packed(const ST* __restrict__ G, ST* __restrict__ E, float* __restrict__ Ebar, const u32x4* __restrict__ Qf,
               const int* __restrict__ Qe, const u32x4* __restrict__ Pf, const int* __restrict__ Pe,
               float* __restrict__ X, float* __restrict__ S1, float* __restrict__ S2, int64_t m, int64_t n, int r,
               int N, OptParams op, int rows_fast) {
  resid_packed_at<OPT, RIGHT, KS, ST>(G, E, Ebar, Qf, Qe, Pf, Pe, X, S1, S2, m, n, r, N, op,
                                      rows_fast ? blockIdx.y : blockIdx.x, rows_fast ? blockIdx.x : blockIdx.y);
}

// Without error feedback (E^(i) and Ebar stay zero): Ghat = P Rbar and the
// optimizer, over 64 x 64 tiles of the m x n layout.  OPT 2: the plain step
// of GaLore, whose Rbar holds its step direction.
template <int OPT, bool RIGHT>
__global__ void __launch_bounds__(256)
k_recon_opt(float* __restrict__ Ebar, const float* __restrict__ Rbar, const float* __restrict__ Ut,
            const int* __restrict__ J, float* __restrict__ X, float* __restrict__ S1, float* __restrict__ S2,
            int64_t m, int64_t n, int64_t d, int64_t D, int r, OptParams op) {
  constexpr int ROWS = 64, COLS = 64;
  using T = MfmaTile<ROWS, COLS, 2, 2>;
  static_assert(T::TM == 1 && T::TN == 1, "one block per wave");
  __shared__ __align__(16) float smem[T::LDS_FLOATS];
  const int c0 = blockIdx.x * COLS, r0 = blockIdx.y * ROWS;
  T tile;
  if (!RIGHT) {
    // rows a < d, columns b < D: C[a][b] = sum_k Ut[J[k]][a] Rbar[k][b]
    LoadR<ROWS, 32, false, true> la(Ut, nullptr, d, r0, (int)d, r, J);
    LoadR<COLS, 32, false> lb(Rbar, nullptr, D, c0, (int)D, r);
    tile.run(la, lb, r, smem);
  } else {
    // rows b < D, columns a < d: C[b][a] = sum_k Rbar[k][b] Ut[J[k]][a]
    LoadR<ROWS, 32, false> la(Rbar, nullptr, D, r0, (int)D, r);
    LoadR<COLS, 32, false, true> lb(Ut, nullptr, d, c0, (int)d, r, J);
    tile.run(la, lb, r, smem);
  }
  const uint32_t bytes = (uint32_t)(m * n * 4);
  const BufRsrc Xr = buf_rsrc(X, bytes), S1r = buf_rsrc(S1, bytes), Ebr = buf_rsrc(Ebar, bytes);
  const BufRsrc S2r = buf_rsrc(OPT == 1 ? S2 : S1, bytes);
  const int64_t cc = c0 + tile.col(0);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int64_t row = r0 + tile.row(0, v);
    const uint32_t o = (cc < n && row < m) ? (uint32_t)((row * n + cc) * 4) : kBufNone;
    const float gh = tile.acc[0][0][v];
    float xv = buf_ld(Xr, o);
    if (OPT == 2) {
      xv = xv - op.lr * gh;
    } else {
      float s1 = buf_ld(S1r, o);
      s1 = op.beta1 * s1 + (1.0f - op.beta1) * gh;
      if (OPT == 0) {
        xv = xv - op.lr * s1;
      } else {
        float s2 = buf_ld(S2r, o);
        s2 = op.beta2 * s2 + (1.0f - op.beta2) * gh * gh;
        xv = xv - op.lr * s1 / (sqrtf(s2) + op.eps);
        buf_st(S2r, o, s2);
      }
      buf_st(S1r, o, s1);
    }
    buf_st(Ebr, o, 0.0f);
    buf_st(Xr, o, xv);
  }
}

// S5 + S7 + S8 from fp32 Q^(i) (above rank 256, and where the packed pieces
// would take too much memory), the workers side by side: one 64 x 64 output
// tile of the m x n layout per workgroup (a 32 x 32 MFMA block per wave).
// Each k-slice of P (gathered rows of U^T) is staged once and multiplied
// with the slices of Q^(w) of up to kNW workers into one accumulator per
// worker, so that the MFMAs run back to back over the whole rank-r
// contraction.  Then E^(w) <- (G^(w) - P Q^(w)) + E^(w) for each worker,
// Ghat = (1/N) sum_w P Q^(w) (= P Rbar by linearity, with no product of its
// own), Ebar = the mean of the stored residuals and the optimizer on X.  More than kNW workers take several
// groups (MULTI), the products of the earlier groups summed in registers.
constexpr int kNW = 4;
constexpr int kNWTile = 64;
// the products of one k-slice for all kNW workers of a group, with no branch
// between the MFMAs, so that the LDS reads of the unrolled loop are issued
// ahead of them (a branch per worker made every MFMA wait for its own operand
// read).  The slices of workers beyond N are zero in LDS, so their products
// are zero.
template <bool RIGHT, int BK, int SL, int PT>
__device__ __forceinline__ void nw_slice(const float* smem, int soff, int qoff, int kh, f32x16 (&acc)[kNW]) {
#pragma unroll
  for (int kk = 0; kk < BK / 2; ++kk) {
    const int row = (2 * kk + kh) * PT;
    const float sv = smem[row + soff];
#pragma unroll
    for (int w = 0; w < kNW; ++w) {
      const float qw = smem[(1 + w) * SL + row + qoff];
      acc[w] = RIGHT ? mfma32(qw, sv, acc[w]) : mfma32(sv, qw, acc[w]);
    }
  }
}
// VEC: the operand slices load through buffer descriptors as float4s (d and
// D multiples of 4, U^T and every group's Q within 2^31 bytes)
template <int OPT, bool RIGHT, bool MULTI, class ST, bool VEC>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_resid_nw(const ST* __restrict__ G, ST* __restrict__ E, float* __restrict__ Ebar,
           const float* __restrict__ Mbar, const float* __restrict__ Q, const float* __restrict__ Ut,
           const int* __restrict__ J, float* __restrict__ X, float* __restrict__ S1, float* __restrict__ S2,
           int64_t m, int64_t n, int64_t d, int64_t D, int r, int N, OptParams op, int rows_fast) {
  constexpr int BK = 32, T = kNWTile;
  constexpr int PT = T + 4, SL = BK * PT;        // LDS pitch and slice size (P, then one per worker)
  __shared__ __align__(16) float smem[(1 + kNW) * SL];
  const int lane = lane_id(), wv = wave_id();
  const int wm = wv >> 1, wn = wv & 1;
  const int kh = lane >> 5, l32 = lane & 31;
  // row tiles are the fast index: the workgroups in flight share the Q
  // slices of a few column tiles, so that each XCD's L2 holds them (and its
  // rows of P) instead of every row tile streaming all of Q again (columns
  // fast only when the column tiles exceed the grid's y extent)
  const int r0 = (rows_fast ? blockIdx.x : blockIdx.y) * T, c0 = (rows_fast ? blockIdx.y : blockIdx.x) * T;
  const int s0 = RIGHT ? c0 : r0, q0 = RIGHT ? r0 : c0;   // first P row / first Q column of the tile
  // the P operand is the MFMA's A (left: tile rows) or B (right: tile columns)
  const int soff = (RIGHT ? wn : wm) * 32 + l32, qoff = (RIGHT ? wm : wn) * 32 + l32;
  const int64_t mn = m * n;
  const uint32_t bytes = (uint32_t)(mn * 4);
  const int64_t col = c0 + wn * 32 + l32;
  float gs[MULTI ? 16 : 1];
  if (MULTI) {
#pragma unroll
    for (int v = 0; v < 16; ++v) gs[MULTI ? v : 0] = 0.f;
  }
  float esum[16];   // the stored residuals' sum over the workers (for Ebar)
#pragma unroll
  for (int v = 0; v < 16; ++v) esum[v] = 0.f;
  f32x16 acc[kNW];
  const int64_t rD = (int64_t)r * D;
  const int nk = (r + BK - 1) / BK;
  for (int w0 = 0; w0 < N; w0 += kNW) {
    const int nw = N - w0 < kNW ? N - w0 : kNW;
#pragma unroll
    for (int w = 0; w < kNW; ++w)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[w][v] = 0.f;
    // one loader per worker slot, each loading into registers of its own, so
    // that the loads of all slots are in flight together (one loader moved
    // from slot to slot made each slot's loads wait for the previous slot's
    // to land); a slot beyond N reads nothing (contraction length 0).  VEC:
    // buffer loads through one descriptor for U^T and one for this group's Q.
    static_assert(kNW == 4, "one loader per worker slot");
    using LS = std::conditional_t<VEC, LoadRB<T, BK, true>, LoadR<T, BK, false, true>>;
    using LQ = std::conditional_t<VEC, LoadRB<T, BK, false>, LoadR<T, BK, false>>;
    const BufRsrc ur = buf_rsrc(Ut, VEC ? (uint32_t)(d * d * 4) : 0u);
    const BufRsrc qr = buf_rsrc(Q + (int64_t)w0 * rD, VEC ? (uint32_t)(nw * rD * 4) : 0u);
    auto make_s = [&]() {
      if constexpr (VEC) return LS(ur, 0u, (int)d, s0, (int)d, r, J);
      else return LS(Ut, nullptr, d, s0, (int)d, r, J);
    };
    auto slot = [&](int w) {
      if constexpr (VEC) return LQ(qr, (uint32_t)((w < nw ? w : 0) * rD * 4), (int)D, q0, (int)D, w < nw ? r : 0);
      else return LQ(Q + (int64_t)(w0 + (w < nw ? w : 0)) * rD, nullptr, D, q0, (int)D, w < nw ? r : 0);
    };
    LS ls = make_s();
    LQ lq[kNW] = {slot(0), slot(1), slot(2), slot(3)};
    auto fetch = [&](int k0) {
      ls.fetch(k0);
#pragma unroll
      for (int w = 0; w < kNW; ++w) lq[w].fetch(k0);
    };
    auto put = [&]() {
      ls.template put<PT>(smem);
#pragma unroll
      for (int w = 0; w < kNW; ++w) lq[w].template put<PT>(smem + (1 + w) * SL);
    };
    fetch(0);
    put();
    __syncthreads();
    for (int kb = 0; kb < nk; ++kb) {
      const bool more = kb + 1 < nk;
      if (more) fetch((kb + 1) * BK);
      nw_slice<RIGHT, BK, SL, PT>(smem, soff, qoff, kh, acc);
      __syncthreads();
      if (more) {
        put();
        __syncthreads();
      }
    }
    // the residuals of this group's workers
#pragma unroll
    for (int w = 0; w < kNW; ++w) {
      if (w >= nw) break;
      const BufRsrc Gw = buf_rsrc_s(G + (int64_t)(w0 + w) * mn, mn);
      const BufRsrc Ew = buf_rsrc_s(E + (int64_t)(w0 + w) * mn, mn);
      uint32_t ob[16];
      float gv[16], eo[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t row = r0 + wm * 32 + mfma32_row(v, lane);
        ob[v] = (row < m && col < n) ? (uint32_t)((row * n + col) * 4) : kBufNone;
        gv[v] = buf_lde<ST>(Gw, ob[v]);
        eo[v] = buf_lde<ST>(Ew, ob[v]);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        // (G - P Q) + E: G and P Q nearly cancel, E is the small part
        const float e = (gv[v] - acc[w][v]) + eo[v];
        buf_ste<ST>(Ew, ob[v], e);
        esum[v] += stored<ST>(e);
        if (MULTI) gs[MULTI ? v : 0] += acc[w][v];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const float inv_n = 1.0f / (float)N;
  const BufRsrc Xr = buf_rsrc(X, bytes), S1r = buf_rsrc(S1, bytes), Ebr = buf_rsrc(Ebar, bytes);
  const BufRsrc S2r = buf_rsrc(OPT == 1 ? S2 : S1, bytes);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int64_t row = r0 + wm * 32 + mfma32_row(v, lane);
    const uint32_t o = (row < m && col < n) ? (uint32_t)((row * n + col) * 4) : kBufNone;
    // workers beyond N hold zero products
    float sum = MULTI ? gs[MULTI ? v : 0] : acc[0][v];
    if (!MULTI) {
#pragma unroll
      for (int w = 1; w < kNW; ++w) sum += acc[w][v];
    }
    const float gh = sum * inv_n;
    float xv = buf_ld(Xr, o);
    float s1 = buf_ld(S1r, o);
    if (OPT == 0) {
      s1 = op.beta1 * s1 + (1.0f - op.beta1) * gh;
      xv = xv - op.lr * s1;
    } else {
      float s2 = buf_ld(S2r, o);
      s1 = op.beta1 * s1 + (1.0f - op.beta1) * gh;
      s2 = op.beta2 * s2 + (1.0f - op.beta2) * gh * gh;
      xv = xv - op.lr * s1 / (sqrtf(s2) + op.eps);
      buf_st(S2r, o, s2);
    }
    buf_st(S1r, o, s1);
    buf_st(Ebr, o, esum[v] * inv_n);
    buf_st(Xr, o, xv);
    if ((v & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
}

template <class ST>
static hipError_t launch_resid_opt_st(const MatView& v, const OptParams& o, hipStream_t s) {
  const ST* G = static_cast<const ST*>(v.G);
  ST* E = static_cast<ST*>(v.E);
  const dim3 grid((unsigned)((v.n + 63) / 64), (unsigned)((v.m + 63) / 64));
  if (v.packed) {
    // column tiles on x: rows of tiles in flight read whole rows of G and E.  A
    // left-sided matrix then streams Q once a row of tiles (33 GB at 8192 x 28672
    // where 18 would do), but mostly from the memory-side cache: row tiles on x,
    // which keep Q's slices in the L2s, measured 5.39 ms there against 5.29, 418
    // us at 4096 x 4096 against 380, 1.10 ms at 4096 x 11008 in bf16 against 1.05.
    // Row tiles on x only when they exceed a grid's y extent (65535: m above
    // 4194240; the column tiles are few then, m n being below 2^30)
    const int rows_fast = grid.y > 65535u ? 1 : 0;
    const dim3 gp = rows_fast ? dim3(grid.y, grid.x) : grid;
#define GLR_RP(OPT, R, KS)                                                                                  \
  hipLaunchKernelGGL((k_resid_packed<OPT, R, KS, ST>), gp, dim3(kThreads), 0, s, G, E, v.Ebar,              \
                     (const u32x4*)v.Qf, v.Qe, (const u32x4*)v.Pf, v.Pe, v.X, v.S1, v.S2, v.m, v.n, v.r, v.N, \
                     o, rows_fast)
#define GLR_RP2(OPT, R)                       \
  switch (pack_steps(v.r)) {                  \
    case 1: GLR_RP(OPT, R, 1); break;         \
    case 2: GLR_RP(OPT, R, 2); break;         \
    case 4: GLR_RP(OPT, R, 4); break;         \
    case 8: GLR_RP(OPT, R, 8); break;         \
    default: GLR_RP(OPT, R, 16);              \
  }
    if (o.opt == 0)      { if (v.right) { GLR_RP2(0, true) } else { GLR_RP2(0, false) } }
    else if (o.opt == 1) { if (v.right) { GLR_RP2(1, true) } else { GLR_RP2(1, false) } }
    else return hipErrorInvalidValue;
#undef GLR_RP2
#undef GLR_RP
    return hipGetLastError();
  }
  if (o.ef) {
    // without packed operands (above rank 256, or packed_resid): one fused pass
    // with the workers side by side
    const bool multi = v.N > kNW;
    const unsigned rt = (unsigned)((v.m + kNWTile - 1) / kNWTile), ct = (unsigned)((v.n + kNWTile - 1) / kNWTile);
    const int rows_fast = ct <= 65535u ? 1 : 0;
    dim3 gw(rows_fast ? rt : ct, rows_fast ? ct : rt);
    // the conditions of the buffer loaders: float4 rows, and U^T and one
    // group's Q within 2^31 bytes
    const bool vec = v.d % 4 == 0 && v.D % 4 == 0 && (reinterpret_cast<uintptr_t>(v.Ut) & 3) == 0 &&
                     (reinterpret_cast<uintptr_t>(v.Q) & 3) == 0 && v.d * v.d * 4 < ((int64_t)1 << 31) &&
                     (int64_t)kNW * v.r * v.D * 4 < ((int64_t)1 << 31);
#define GLR_RW(OPT, R, MU)                                                                                   \
  do {                                                                                                       \
    if (vec)                                                                                                 \
      hipLaunchKernelGGL((k_resid_nw<OPT, R, MU, ST, true>), gw, dim3(kThreads), 0, s, G, E, v.Ebar, v.Mbar,  \
                         v.Q, v.Ut, v.J, v.X, v.S1, v.S2, v.m, v.n, v.d, v.D, v.r, v.N, o, rows_fast);       \
    else                                                                                                     \
      hipLaunchKernelGGL((k_resid_nw<OPT, R, MU, ST, false>), gw, dim3(kThreads), 0, s, G, E, v.Ebar, v.Mbar, \
                         v.Q, v.Ut, v.J, v.X, v.S1, v.S2, v.m, v.n, v.d, v.D, v.r, v.N, o, rows_fast);       \
  } while (0)
#define GLR_RW2(OPT, R) do { if (multi) GLR_RW(OPT, R, true); else GLR_RW(OPT, R, false); } while (0)
    if (o.opt == 0)      { if (v.right) GLR_RW2(0, true); else GLR_RW2(0, false); }
    else if (o.opt == 1) { if (v.right) GLR_RW2(1, true); else GLR_RW2(1, false); }
    else return hipErrorInvalidValue;
#undef GLR_RW2
#undef GLR_RW
    return hipGetLastError();
  }
#define GLR_RO(OPT, R)                                                                                            \
  hipLaunchKernelGGL((k_recon_opt<OPT, R>), grid, dim3(kThreads), 0, s, v.Ebar, v.Rbar, v.Ut, v.J, v.X, v.S1, v.S2, \
                     v.m, v.n, v.d, v.D, v.r, o)
  if (o.opt == 0)      { if (v.right) GLR_RO(0, true); else GLR_RO(0, false); }
  else if (o.opt == 1) { if (v.right) GLR_RO(1, true); else GLR_RO(1, false); }
  else if (sizeof(ST) == 2) return hipErrorInvalidValue;   // GaLore runs on fp32 storage only
  else { if (v.right) GLR_RO(2, true); else GLR_RO(2, false); }
#undef GLR_RO
  return hipGetLastError();
}
hipError_t launch_resid_opt(const MatView& v, const OptParams& o, hipStream_t s) {
  return v.st16 ? launch_resid_opt_st<bf16_t>(v, o, s) : launch_resid_opt_st<float>(v, o, s);
}

// Algorithm 5 (distributed Adam-type GaLore): the Adam moments live in the
// r x D subspace (S1 = M, S2 = V, row-major r x D, oriented) and restart from
// zero at every refresh; the step direction Rhat = M / (sqrt(V) + eps)
// replaces Rbar, so that the reconstruction P Rhat and X -= lr P Rhat follow
// in k_recon_opt<2>.  Moments in the main text's form (eq-adam).
__global__ void k_galore_adam(float* __restrict__ Rbar, float* __restrict__ S1, float* __restrict__ S2, int64_t n,
                              float beta1, float beta2, float eps, int reset) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride) {
    const float g = Rbar[i];
    const float m0 = reset ? 0.0f : S1[i], v0 = reset ? 0.0f : S2[i];
    const float m1 = beta1 * m0 + (1.0f - beta1) * g;
    const float v1 = beta2 * v0 + (1.0f - beta2) * g * g;
    S1[i] = m1;
    S2[i] = v1;
    Rbar[i] = m1 / (sqrtf(v1) + eps);
  }
}

hipError_t launch_galore_adam(const MatView& v, const OptParams& o, bool reset, hipStream_t s) {
  const int64_t n = (int64_t)v.r * v.D;
  hipLaunchKernelGGL(k_galore_adam, dim3(grid_for(n)), dim3(256), 0, s, v.Rbar, v.S1, v.S2, n, o.beta1, o.beta2,
                     o.eps, reset ? 1 : 0);
  return hipGetLastError();
}

// Algorithm 3 at a refresh step: E^(i) = 0, Ebar = 0, Ghat = Mbar.
template <int OPT, class ST>
__global__ void k_full_refresh(const float* __restrict__ Mbar, ST* __restrict__ E,
                               float* __restrict__ Ebar, float* __restrict__ X,
                               float* __restrict__ S1, float* __restrict__ S2, int64_t mn, int N,
                               OptParams op) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < mn; i += stride) {
    const float gh = Mbar[i];
    for (int w = 0; w < N; ++w) E[(int64_t)w * mn + i] = ST(0);
    Ebar[i] = 0.f;
    float x = X[i];
    if (OPT == 0) {
      const float mm = op.beta1 * S1[i] + (1.0f - op.beta1) * gh;
      S1[i] = mm;
      x = x - op.lr * mm;
    } else {
      const float m1 = op.beta1 * S1[i] + (1.0f - op.beta1) * gh;
      const float m2 = op.beta2 * S2[i] + (1.0f - op.beta2) * gh * gh;
      S1[i] = m1;
      S2[i] = m2;
      x = x - op.lr * m1 / (sqrtf(m2) + op.eps);
    }
    X[i] = x;
  }
}

template <class ST>
static hipError_t launch_full_refresh_st(const MatView& v, const OptParams& o, hipStream_t s) {
  const int64_t mn = v.m * v.n;
  ST* E = static_cast<ST*>(v.E);
  if (o.opt == 0)
    hipLaunchKernelGGL((k_full_refresh<0, ST>), dim3(grid_for(mn, 4)), dim3(kThreads), 0, s, v.Mbar, E,
                       v.Ebar, v.X, v.S1, v.S2, mn, v.N, o);
  else
    hipLaunchKernelGGL((k_full_refresh<1, ST>), dim3(grid_for(mn, 4)), dim3(kThreads), 0, s, v.Mbar, E,
                       v.Ebar, v.X, v.S1, v.S2, mn, v.N, o);
  return hipGetLastError();
}
hipError_t launch_full_refresh(const MatView& v, const OptParams& o, hipStream_t s) {
  return v.st16 ? launch_full_refresh_st<bf16_t>(v, o, s) : launch_full_refresh_st<float>(v, o, s);
}


// ---------------------------------------------------------------------------
// Grouped selection step: every kernel of a selection step in one launch over
// all matrices.  Each matrix owns a range of blocks (tables of first blocks);
// a block finds its matrix and runs the per-matrix body with the coordinates
// it has in that matrix's own launch, so each matrix computes exactly what its
// own launches compute.  Many small matrices then fill the chip together
// instead of a few CUs each.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int group_find(const int* __restrict__ first, int num, int b) {
  int lo = 0, hi = num - 1;   // the last m with first[m] <= b
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// projection tiles of rank r (at most kGroupMaxRank): BM x BN, WM x WN waves,
// fp64 flush of the slices (false: the split product)
#define GLR_PROJ_TIERS(X)                                   \
  if (r <= 32) X(32, 128, 1, 4, true);                      \
  else if (r <= kProjFlushRank) X(64, 64, 2, 2, true);      \
  else X(128, 64, 2, 2, false)

template <class ST>
__global__ void k_g_ef_mean(const GroupMat* __restrict__ gm, const int* __restrict__ first, int num, int check) {
  const int m = group_find(first, num, blockIdx.x);
  const MatView& v = gm[m].v;
  ef_mean_at(static_cast<const ST*>(v.G), v.Ebar, v.Mbar, v.m * v.n, v.N, v.status, check, v.amax,
             blockIdx.x - first[m], first[m + 1] - first[m]);
}

template <int BT, bool RIGHT, bool APPROX, bool BF16>
__global__ void __launch_bounds__(256, BT == 64 ? 4 : 2)
k_g_sel_scores(const GroupMat* __restrict__ gm, const int* __restrict__ first, int num, uint32_t tstep,
               uint32_t key0, uint32_t key1) {
  const int m = group_find(first, num, blockIdx.x);
  const MatView& v = gm[m].v;
  const int local = blockIdx.x - first[m], gx = (int)((v.d + BT - 1) / BT);
  sel_scores_at<BT, RIGHT, APPROX, BF16>(v.Mbar, v.Ut, v.d, v.D, v.lam_part, (uint32_t)v.mat, tstep, key0, key1,
                                     v.amax, v.umax, local % gx, local / gx);
}

// (each matrix's workgroup folds its own partials, whatever their count: a
// selection step of four 2048 x 2048 matrices, 65536 partials each, takes 488 us
// so and 498 with a fold over the chip before it; four 2048 x 8192, 262144, the
// same; two 2048 x 28672, 917504, 3.41 and 3.36 ms)
__global__ void __launch_bounds__(kToprThreads)
k_g_topr(const GroupMat* __restrict__ gm, int approx) {
  const MatView& v = gm[blockIdx.x].v;
  topr_at(v.lam_part, (int)((v.D + 63) / 64), true, approx, (int)v.d, v.score, v.r, v.J);
}

template <int BM, int BN, int WM, int WN, bool RIGHT, bool FLUSH, class ST>
__global__ void __launch_bounds__(256, FLUSH ? 1 : 2)
k_g_proj(const GroupMat* __restrict__ gm, const int* __restrict__ first, int num) {
  const int m = group_find(first, num, blockIdx.x);
  const GroupMat& g = gm[m];
  const MatView& v = g.v;
  const int gx = (int)((v.D + BN - 1) / BN), gy = (v.r + BM - 1) / BM;
  const int local = blockIdx.x - first[m], rest = local / gx;
  if constexpr (FLUSH)
    proj_at<BM, BN, WM, WN, RIGHT, ST>(static_cast<const ST*>(v.G), static_cast<const ST*>(v.E), v.Ut, v.J,
                                             v.Qpart, v.d, v.D, v.r, v.N, g.kslice, local % gx, rest % gy, rest / gy);
  else
    proj_split_at<BM, WM, WN, RIGHT, ST>(static_cast<const ST*>(v.G), static_cast<const ST*>(v.E), v.Ut, v.J, v.Qpart,
                                         v.d, v.D, v.r, v.N, g.kslice, local % gx, rest % gy, rest / gy);
}

template <int KS>
__global__ void __launch_bounds__(kThreads)
k_g_pack_waves(const GroupMat* __restrict__ gm, const int* __restrict__ first, int num) {
  const int m = group_find(first, num, blockIdx.x);
  const GroupMat& g = gm[m];
  const MatView& v = g.v;
  pack_waves<KS>(v.Qpart, g.splits, v.N, v.r, v.d, v.D, v.Ut, v.J, (u32x4*)v.Qf, v.Qe, (u32x4*)v.Pf, v.Pe, v.Rbar,
                 blockIdx.x - first[m]);
}

template <int OPT, bool RIGHT, int KS, class ST>
__global__ void __launch_bounds__(256, KS <= 4 ? 3 : 2)
k_g_resid(const GroupMat* __restrict__ gm, const int* __restrict__ first, int num, OptParams op) {
  const int m = group_find(first, num, blockIdx.x);
  const MatView& v = gm[m].v;
  const int local = blockIdx.x - first[m], gx = (int)((v.n + 63) / 64);
  resid_packed_at<OPT, RIGHT, KS, ST>(static_cast<const ST*>(v.G), static_cast<ST*>(v.E), v.Ebar, (const u32x4*)v.Qf,
                                      v.Qe, (const u32x4*)v.Pf, v.Pe, v.X, v.S1, v.S2, v.m, v.n, v.r, v.N, op, local % gx,
                                      local / gx);
}

void group_fill(GroupMat& g, int (&blocks)[kGrpKinds]) {
  const MatView& v = g.v;
  const int r = v.r;
  g.splits = proj_splits(v.d, v.D, r, v.N);
  g.kslice = proj_kslice(v.d, v.D, r, v.N);
  blocks[kGrpEfMean] = ef_mean_blocks(v.m * v.n);
  blocks[kGrpSel128] = sel_tiles(v.d, v.D, 128);
  blocks[kGrpSel64] = sel_tiles(v.d, v.D, 64);
  int proj = 0;
#define GLR_PROJ_BLOCKS(BM, BN, WM, WN, FL) proj = (int)(((v.D + BN - 1) / BN) * ((r + BM - 1) / BM) * v.N * g.splits)
  GLR_PROJ_TIERS(GLR_PROJ_BLOCKS);
#undef GLR_PROJ_BLOCKS
  blocks[kGrpProj] = proj;
  blocks[kGrpRbar] = pack_blocks(v.d, v.D, v.N, r);
  blocks[kGrpResid] = (int)(((v.n + 63) / 64) * ((v.m + 63) / 64));
}

template <class ST>
static hipError_t launch_group_select_st(const GroupPlan& gp, bool check_finite, bool approx, bool bf16,
                                         uint64_t seed, int64_t t, const OptParams& o, int part, hipStream_t s) {
  if (bf16 && !approx) return hipErrorInvalidValue;
  const int num = gp.num, r = gp.r;
  const bool right = gp.right;
  auto table = [&](int kind) { return gp.first + (int64_t)kind * (num + 1); };
  auto grid = [&](int kind) { return dim3((unsigned)gp.total[kind]); };
  if (part != 2)
    hipLaunchKernelGGL(k_g_ef_mean<ST>, grid(kGrpEfMean), dim3(kThreads), 0, s, gp.gm, table(kGrpEfMean), num,
                       check_finite ? 1 : 0);
  if (part == 1) return hipGetLastError();
  const uint32_t k0 = (uint32_t)(seed & 0xFFFFFFFFu), k1 = (uint32_t)(seed >> 32);
  const uint32_t tt = (uint32_t)((uint64_t)t & 0xFFFFFFFFu);
  const bool few = gp.total[kGrpSel128] < kSelFew;
#define GLR_GSEL1(T, K, R, A, B) \
  hipLaunchKernelGGL((k_g_sel_scores<T, R, A, B>), grid(K), dim3(kThreads), 0, s, gp.gm, table(K), num, tt, k0, k1)
#define GLR_GSEL(R, A, B)                            \
  do {                                               \
    if (few) GLR_GSEL1(64, kGrpSel64, R, A, B);      \
    else GLR_GSEL1(128, kGrpSel128, R, A, B);        \
  } while (0)
  if (right) {
    if (bf16) GLR_GSEL(true, true, true);
    else if (approx) GLR_GSEL(true, true, false);
    else GLR_GSEL(true, false, false);
  } else {
    if (bf16) GLR_GSEL(false, true, true);
    else if (approx) GLR_GSEL(false, true, false);
    else GLR_GSEL(false, false, false);
  }
#undef GLR_GSEL
#undef GLR_GSEL1
  hipLaunchKernelGGL(k_g_topr, dim3((unsigned)num), dim3(kToprThreads), 0, s, gp.gm, approx ? 1 : 0);
#define GLR_GPROJ(BM, BN, WM, WN, FL)                                                                       \
  do {                                                                                                      \
    if (right)                                                                                              \
      hipLaunchKernelGGL((k_g_proj<BM, BN, WM, WN, true, FL, ST>), grid(kGrpProj), dim3(kThreads), 0, s,    \
                         gp.gm, table(kGrpProj), num);                                                      \
    else                                                                                                    \
      hipLaunchKernelGGL((k_g_proj<BM, BN, WM, WN, false, FL, ST>), grid(kGrpProj), dim3(kThreads), 0, s,   \
                         gp.gm, table(kGrpProj), num);                                                      \
  } while (0)
  GLR_PROJ_TIERS(GLR_GPROJ);
#undef GLR_GPROJ
  switch (pack_steps(r)) {
    case 1: hipLaunchKernelGGL(k_g_pack_waves<1>, grid(kGrpRbar), dim3(kThreads), 0, s, gp.gm, table(kGrpRbar), num); break;
    case 2: hipLaunchKernelGGL(k_g_pack_waves<2>, grid(kGrpRbar), dim3(kThreads), 0, s, gp.gm, table(kGrpRbar), num); break;
    case 4: hipLaunchKernelGGL(k_g_pack_waves<4>, grid(kGrpRbar), dim3(kThreads), 0, s, gp.gm, table(kGrpRbar), num); break;
    default: hipLaunchKernelGGL(k_g_pack_waves<8>, grid(kGrpRbar), dim3(kThreads), 0, s, gp.gm, table(kGrpRbar), num);
  }
  static_assert(kGroupMaxRank <= 16 * kPackWaveSteps, "a variant for every rank");
#define GLR_GRO1(OPT, R, KS)                                                                             \
  hipLaunchKernelGGL((k_g_resid<OPT, R, KS, ST>), grid(kGrpResid), dim3(kThreads), 0, s, gp.gm, table(kGrpResid), \
                     num, o)
#define GLR_GRO(OPT, R)                    \
  switch (pack_steps(r)) {                 \
    case 1: GLR_GRO1(OPT, R, 1); break;    \
    case 2: GLR_GRO1(OPT, R, 2); break;    \
    case 4: GLR_GRO1(OPT, R, 4); break;    \
    default: GLR_GRO1(OPT, R, 8);          \
  }
  static_assert(kGroupMaxRank <= 128, "the grouped residual's largest variant");
  if (o.opt == 0) { if (right) { GLR_GRO(0, true) } else { GLR_GRO(0, false) } }
  else            { if (right) { GLR_GRO(1, true) } else { GLR_GRO(1, false) } }
#undef GLR_GRO1
#undef GLR_GRO
  return hipGetLastError();
}
hipError_t launch_group_select(const GroupPlan& gp, bool check_finite, bool approx, bool bf16, uint64_t seed,
                               int64_t t, const OptParams& o, int part, hipStream_t s) {
  return gp.st16 ? launch_group_select_st<bf16_t>(gp, check_finite, approx, bf16, seed, t, o, part, s)
                 : launch_group_select_st<float>(gp, check_finite, approx, bf16, seed, t, o, part, s);
}

}  // namespace glr
