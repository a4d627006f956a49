// Offline table construction for one layer: T = P B (§2.2), then 8-bit block
// floating point quantization (§1).  Not on the inference hot path; it turns
// prototypes and weights into the tables the hot path reads.
//
// T[c][k][m] = sum_d P[c][k][d] * B[d][m] is a double sum over d ascending;
// the products of two fp32 values are exact in double and the library is
// built with -ffp-contract=off, so every entry is one well-defined double.
//
// Quantization of codebook c over its 16 x M entries:
//   offset o_c = (float)((min + max) / 2),  r_c = max |T - o_c|,
//   e_c        = smallest e in [-126, 127] with r_c <= 127 * 2^e,
//   e_c       <- max(e_c, max_c' e_c' - cap)   (127 * C * 2^cap < 2^24),
//   q          = round-half-even((T - o_c) * 2^-e_c),  |q| <= 127.
// T = P B takes four launches: the range of every (codebook, column tile),
// parked in the tile's own part of the codes; per codebook the offset and the
// exponent (parked in scale_out as an integer); the codes; the scales.  (Three
// for small tables: range and exponent in one.)  The entries are evaluated in
// the first and the third (no workspace for a double copy of T).  A given table
// T takes three: statistics (one workgroup per codebook), codes, scales.
//
// Zero prototype columns.  P[c] is zero outside codebook c's subspace, so most
// terms are a zero times a finite weight.  A sum that starts at +0 is never
// -0 and adding +-0 to it changes nothing, so a column d with P[c][k][d] = 0
// for all 16 k is skipped with the sum's bits unchanged, as long as every
// B[d][m] is finite (0 * inf and 0 * NaN are NaN).  Each workgroup lists the
// columns of its codebook that are not all zero, ascending, and the weights
// are checked on the way: every (codebook, tile) checks its share of B's rows.
// One non-finite weight anywhere, and every column is taken (for the fp32 table,
// whose columns do not depend on each other, by the tiles that hold one).
//
// Bound: launches and latency (P and B once from HBM, a few columns per
// codebook); with prototypes that have no zero column, the fp64 FMA rate.
// 128 codebooks, D 1024, M 4096 (8 nonzero columns per codebook): 50 us a build
// against 14.2 ms with every column taken and one workgroup per codebook.
#include "internal.hpp"

#include <type_traits>

namespace mdn {

constexpr int kBuildThreads = 256;
// the statistics pass: one workgroup of kStatsThreads per codebook, kStatsILP
// entries of a thread evaluated together (their sums are independent chains,
// each in its own order)
constexpr int kStatsThreads = 1024;
constexpr int kStatsILP = 4;

constexpr int kChunk = 512;   // prototype columns listed at a time
constexpr int kAllColumns = 4;   // up to so many are all taken: the weights need no look then

// What a workgroup of kBuildThreads keeps of one chunk of P[c]: the columns
// that are not all zero, ascending, and their 16 values (as doubles: they are
// read once per column of the tile).
struct TileLds {
  double p[kChunk][kK];
  int d[kChunk];
  int cnt[2 * kBuildThreads / 64];
  int each[kBuildThreads / 64];   // whether a wavefront takes every column
};

// A tile of T from column col0 of codebook c, all 16 prototypes: a thread has
// KPT of them from k0() and CPT columns colof(j), t[k][j] their sums over d
// ascending.  The product of two floats is exact in double, so the fused
// multiply-add rounds exactly as a multiply and an add do.  `dense` takes the
// zero columns too.  Columns past M read column M - 1.
template <int CPT, bool VEC, int KPT>
struct Tile {
  static constexpr int kCpt = CPT, kKpt = KPT;
  static constexpr bool kVec = VEC;
  static constexpr int kAcross = kBuildThreads * KPT / kK;   // threads side by side
  static constexpr int kCols = CPT * kAcross;
  static __device__ __forceinline__ int k0() { return (int)threadIdx.x / kAcross * KPT; }
  static __device__ __forceinline__ int colof(int col0, int j) {
    const int x = (int)threadIdx.x % kAcross;
    return VEC ? col0 + CPT * x + j : col0 + x + j * kAcross;
  }
  // whether a weight of rows d0 .. d1 in the tile's columns, as far as this
  // thread looks (the threads of a column share its rows), is not finite
  static __device__ __forceinline__ bool not_finite(const float* __restrict__ B, int64_t d0, int64_t d1, int M,
                                                    int col0) {
    bool bad = false;
#pragma unroll 8
    for (int64_t d = d0 + threadIdx.x / kAcross; d < d1; d += kK / KPT)
#pragma unroll
      for (int j = 0; j < CPT; ++j) bad |= !__builtin_isfinite(B[d * M + min(colof(col0, j), M - 1)]);
    return bad;
  }
  // EACH: `dense` differs between threads, and one is enough (asked of all of
  // them once the first prototypes have been requested).
  template <bool EACH = false>
  static __device__ void sums(const float* __restrict__ P, const float* __restrict__ B, int D, int M, int c, int col0,
                              bool dense, TileLds& s, double (&t)[KPT][CPT]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NW = kBuildThreads / 64;
#pragma unroll
    for (int k = 0; k < KPT; ++k)
#pragma unroll
      for (int j = 0; j < CPT; ++j) t[k][j] = 0.0;
    const int kt = k0();
    const float* pc = P + (int64_t)c * kK * D;
    const float* b[CPT];
#pragma unroll
    for (int j = 0; j < CPT; ++j) b[j] = B + (VEC ? min(colof(col0, 0), M - CPT) + j : min(colof(col0, j), M - 1));
    for (int d0 = 0; d0 < D; d0 += kChunk) {
      // two columns per thread, their 16 values in registers
      float v[2][kK];
      bool use[2];
      uint64_t mask[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int d = d0 + h * kBuildThreads + tid;
#pragma unroll
        for (int k = 0; k < kK; ++k) v[h][k] = d < D ? pc[(int64_t)k * D + d] : 0.0f;
      }
      // the previous chunk's (or tile's) list has been read
      if constexpr (EACH) {
        const bool any = __ballot(dense) != 0;
        if (lane == 0) s.each[wave] = any;
      }
      __syncthreads();
      if constexpr (EACH)
#pragma unroll
        for (int w = 0; w < NW; ++w) dense |= s.each[w] != 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        bool nz = dense;
#pragma unroll
        for (int k = 0; k < kK; ++k) nz |= v[h][k] != 0.0f;   // (true for NaN)
        use[h] = nz && d0 + h * kBuildThreads + tid < D;
        mask[h] = __ballot(use[h]);
        if (lane == 0) s.cnt[h * NW + wave] = __popcll(mask[h]);
      }
      __syncthreads();
      int n = 0, at[2] = {0, 0};
#pragma unroll
      for (int i = 0; i < 2 * NW; ++i) {
        if (i < wave) at[0] += s.cnt[i];
        if (i < NW + wave) at[1] += s.cnt[i];
        n += s.cnt[i];
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (use[h]) {
          const int e = at[h] + __popcll(mask[h] & ((1ull << lane) - 1));
          s.d[e] = d0 + h * kBuildThreads + tid;
#pragma unroll
          for (int k = 0; k < kK; ++k) s.p[e][k] = (double)v[h][k];
        }
      __syncthreads();
      // rows of B in flight: 16 / CPT, and 4 for the last 4 and fewer (a block's
      // few columns)
      auto rows = [&](int e0, auto count) {
        constexpr int kU = decltype(count)::value;
        float w[kU][CPT];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int64_t ro = (int64_t)s.d[min(e0 + u, n - 1)] * M;
          if constexpr (VEC) {
            const float4 q = *reinterpret_cast<const float4*>(b[0] + ro);
            w[u][0] = q.x; w[u][1] = q.y; w[u][2] = q.z; w[u][3] = q.w;
          } else {
#pragma unroll
            for (int j = 0; j < CPT; ++j) w[u][j] = b[j][ro];
          }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
          if (e0 + u < n) {
#pragma unroll
            for (int k = 0; k < KPT; ++k) {
              const double pv = s.p[e0 + u][kt + k];
#pragma unroll
              for (int j = 0; j < CPT; ++j) t[k][j] = __fma_rn(pv, (double)w[u][j], t[k][j]);
            }
          }
      };
      int e0 = 0;
      if constexpr (CPT < 4)
        for (; n - e0 > 4; e0 += 16 / CPT) rows(e0, std::integral_constant<int, 16 / CPT>{});
      for (; e0 < n; e0 += 4) rows(e0, std::integral_constant<int, 4>{});
    }
  }
};

// a double at any byte address (the codes are a byte array)
struct __attribute__((packed)) F64u { double v; };

// lo and hi over this thread's entries of a tile
template <class T>
__device__ __forceinline__ void widen(const double (&t)[T::kKpt][T::kCpt], int col0, int M, double& lo, double& hi) {
#pragma unroll
  for (int j = 0; j < T::kCpt; ++j)
    if (T::colof(col0, j) < M)
#pragma unroll
      for (int k = 0; k < T::kKpt; ++k) {
        lo = fmin(lo, t[k][j]);
        hi = fmax(hi, t[k][j]);
      }
}

// lo and hi over the workgroup, for thread 0 (true there); has a barrier
__device__ __forceinline__ bool block_range(double (&s_red)[2][kBuildThreads / 64], double& lo, double& hi) {
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o));
    hi = fmax(hi, __shfl_xor(hi, o));
  }
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = lo;
    s_red[1][threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x != 0) return false;
  for (int w = 1; w < kBuildThreads / 64; ++w) {
    lo = fmin(lo, s_red[0][w]);
    hi = fmax(hi, s_red[1][w]);
  }
  return true;
}

// The range of T over one (codebook, column tile), parked in the first 16
// bytes of the tile's codes ([lo, hi]; a tile of any codebook has at least 16
// bytes).  lo = NaN says that a weight among this workgroup's share of B is
// not finite (a range of entries is never NaN: fmin and fmax skip NaN).
template <class T>
__global__ void __launch_bounds__(kBuildThreads)
build_range_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M, int tiles,
                   int8_t* lut) {
  __shared__ TileLds s;
  __shared__ double s_red[2][kBuildThreads / 64];
  __shared__ int s_bad;
  const int c = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const int col0 = tile * T::kCols;
  if (threadIdx.x == 0) s_bad = 0;
  double t[T::kKpt][T::kCpt];
  T::sums(P, B, D, M, c, col0, false, s, t);   // (has barriers: s_bad is set)
  if (T::not_finite(B, (int64_t)c * D / C, (int64_t)(c + 1) * D / C, M, col0)) s_bad = 1;
  double lo = __builtin_inf(), hi = -__builtin_inf();
  widen<T>(t, col0, M, lo, hi);
  if (block_range(s_red, lo, hi)) {
    F64u* out = reinterpret_cast<F64u*>(lut + (int64_t)c * kK * M + 16 * tile);
    out[0].v = s_bad ? __builtin_nan("") : lo;
    out[1].v = hi;
  }
}

constexpr int kDenseBit = 1 << 16;   // in a parked exponent: take every prototype column

// Offset and exponent of codebook c from its range; r = max |T - o| is taken at
// an end of it (rounding is monotone).
__device__ __forceinline__ void park_exponent(double lo, double hi, bool dense, int c, float* __restrict__ scale_out,
                                              float* __restrict__ offset_out) {
  const float o = (float)__ddiv_rn(__dadd_rn(lo, hi), 2.0);
  const double r = fmax(fmax(0.0, fabs(__dsub_rn(lo, (double)o))), fabs(__dsub_rn(hi, (double)o)));
  int ex = -126;
  while (ex < 127 && r > 127.0 * __builtin_ldexp(1.0, ex)) ++ex;
  offset_out[c] = o;
  // parked, replaced by table_scale_kernel
  reinterpret_cast<int*>(scale_out)[c] = ex + (dense ? kDenseBit : 0);
}

// The same from the ranges of its tiles, c = blockIdx.x.  With a non-finite
// weight anywhere the range is evaluated here over every prototype column, and
// the codes are told to do the same.
template <class T>
__global__ void __launch_bounds__(kBuildThreads)
build_exponent_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M, int tiles,
                      const int8_t* lut, float* __restrict__ scale_out, float* __restrict__ offset_out) {
  __shared__ TileLds s;
  __shared__ double s_red[2][kBuildThreads / 64];
  __shared__ int s_bad;
  const int c = blockIdx.x;
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  for (int e = threadIdx.x; e < C * tiles; e += kBuildThreads) {
    const int8_t* at = lut + (int64_t)(e / tiles) * kK * M + 16 * (e % tiles);
    if (__builtin_isnan(reinterpret_cast<const F64u*>(at)->v)) s_bad = 1;
  }
  __syncthreads();
  const bool dense = s_bad != 0;
  double lo = __builtin_inf(), hi = -__builtin_inf();
  if (!dense) {
    for (int e = threadIdx.x; e < tiles; e += kBuildThreads) {
      const F64u* in = reinterpret_cast<const F64u*>(lut + (int64_t)c * kK * M + 16 * e);
      lo = fmin(lo, in[0].v);
      hi = fmax(hi, in[1].v);
    }
  } else {
    for (int tile = 0; tile < tiles; ++tile) {
      double t[T::kKpt][T::kCpt];
      T::sums(P, B, D, M, c, tile * T::kCols, true, s, t);
      widen<T>(t, tile * T::kCols, M, lo, hi);
    }
  }
  if (block_range(s_red, lo, hi)) park_exponent(lo, hi, dense, c, scale_out, offset_out);
}

// Both in one launch for tables of one tile and few weights: every workgroup
// looks through all of B itself.
template <class T>
__global__ void __launch_bounds__(kBuildThreads)
build_small_exponent_kernel(const float* __restrict__ P, const float* __restrict__ B, int D, int M,
                            float* __restrict__ scale_out, float* __restrict__ offset_out) {
  __shared__ TileLds s;
  __shared__ double s_red[2][kBuildThreads / 64];
  const int c = blockIdx.x;
  const bool dense = D <= kAllColumns || __syncthreads_or(T::not_finite(B, 0, D, M, 0));
  double t[T::kKpt][T::kCpt];
  T::sums(P, B, D, M, c, 0, dense, s, t);
  double lo = __builtin_inf(), hi = -__builtin_inf();
  widen<T>(t, 0, M, lo, hi);
  if (block_range(s_red, lo, hi)) park_exponent(lo, hi, dense, c, scale_out, offset_out);
}

__device__ __forceinline__ int parked_exponent(int v) { return v >= kDenseBit / 2 ? v - kDenseBit : v; }

__device__ __forceinline__ int8_t code_of(double t, double o, double inv) {
  return (int8_t)(int)fmin(127.0, fmax(-127.0, rint(__dmul_rn(__dsub_rn(t, o), inv))));
}

__device__ int max_parked_exponent(const float* __restrict__ scale_out, int C, int* s_max);

template <class T>
__global__ void __launch_bounds__(kBuildThreads)
build_codes_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M, int tiles, int cap,
                   const float* __restrict__ scale_out, const float* __restrict__ offset_out,
                   int8_t* __restrict__ lut) {
  __shared__ TileLds s;
  __shared__ int s_max;
  const int c = blockIdx.x / tiles, col0 = (blockIdx.x % tiles) * T::kCols;
  const int parked = reinterpret_cast<const int*>(scale_out)[c];
  double t[T::kKpt][T::kCpt];
  T::sums(P, B, D, M, c, col0, parked >= kDenseBit / 2, s, t);
  const int ex = max(parked_exponent(parked), max_parked_exponent(scale_out, C, &s_max) - cap);
  const double o = (double)offset_out[c], inv = __builtin_ldexp(1.0, -ex);
  int8_t* out = lut + ((int64_t)c * kK + T::k0()) * M;
#pragma unroll
  for (int k = 0; k < T::kKpt; ++k) {
    if constexpr (T::kVec) {   // M % 4 == 0: a thread's 4 columns exist together
      const int m = T::colof(col0, 0);
      if (m < M) {
        uint32_t q = 0;
#pragma unroll
        for (int j = 0; j < T::kCpt; ++j) q |= (uint32_t)(uint8_t)code_of(t[k][j], o, inv) << (8 * j);
        *reinterpret_cast<uint32_t*>(out + (int64_t)k * M + m) = q;
      }
    } else {
#pragma unroll
      for (int j = 0; j < T::kCpt; ++j) {
        const int m = T::colof(col0, j);
        if (m < M) out[(int64_t)k * M + m] = code_of(t[k][j], o, inv);
      }
    }
  }
}

// The fp32 table.  A column that holds a weight that is not finite needs every
// prototype column, and a workgroup with one takes them all.  Few weights
// (SMALL) the workgroup looks through itself; else weights_kernel has, and
// left word j of the 64 columns from 64 i, the bits of 32 of them, in the first
// row of every codebook, at column 64 i + j.
template <class T, bool SMALL>
__global__ void __launch_bounds__(kBuildThreads)
build_f32_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M, int tiles, float* lut) {
  __shared__ TileLds s;
  const int c = blockIdx.x / tiles, col0 = (blockIdx.x % tiles) * T::kCols;
  float* out = lut + ((int64_t)c * kK + T::k0()) * M;
  bool bad = false;
  if constexpr (SMALL) {
    bad = D <= kAllColumns || T::not_finite(B, 0, D, M, col0);
  } else {
    const uint32_t* parked = reinterpret_cast<const uint32_t*>(lut + (int64_t)c * kK * M);
#pragma unroll
    for (int j = 0; j < T::kCpt; ++j) {
      const int m = min(T::colof(col0, j), M - 1);
      bad |= (parked[(m & ~63) + (m >> 5 & 1)] >> (m & 31)) & 1;
    }
  }
  double t[T::kKpt][T::kCpt];
  T::template sums<true>(P, B, D, M, c, col0, bad, s, t);   // (every word has been read before any is replaced)
#pragma unroll
  for (int k = 0; k < T::kKpt; ++k) {
    if constexpr (T::kVec) {
      const int m = T::colof(col0, 0);
      if (m < M)
        *reinterpret_cast<float4*>(out + (int64_t)k * M + m) =
            make_float4((float)t[k][0], (float)t[k][1], (float)t[k][2], (float)t[k][3]);
    } else {
#pragma unroll
      for (int j = 0; j < T::kCpt; ++j) {
        const int m = T::colof(col0, j);
        if (m < M) out[(int64_t)k * M + m] = (float)t[k][j];
      }
    }
  }
}

// Small tables of few weights, an entry per thread and no list.
__global__ void __launch_bounds__(kBuildThreads)
build_f32_small_kernel(const float* __restrict__ P, const float* __restrict__ B, int D, int M, int total,
                       float* __restrict__ lut) {
  const int e = (int)blockIdx.x * kBuildThreads + (int)threadIdx.x;
  if (e >= total) return;
  const int row = e / M, m = e - row * M;
  double t = 0.0;
#pragma unroll 16
  for (int d = 0; d < D; ++d) t = __fma_rn((double)P[row * D + d], (double)B[d * M + m], t);
  lut[e] = (float)t;
}

// Which columns hold a weight that is not finite, 64 of them per workgroup.
constexpr int kWeightThreads = 1024;
__global__ void __launch_bounds__(kWeightThreads)
weights_kernel(const float* __restrict__ B, int C, int D, int M, float* __restrict__ lut) {
  __shared__ int s_bad[64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int m0 = blockIdx.x * 64, m = m0 + lane;
  if (tid < 64) s_bad[tid] = 0;
  __syncthreads();
  bool bad = false;
#pragma unroll 8
  for (int d = tid >> 6; d < D; d += kWeightThreads / 64)
    bad |= !__builtin_isfinite(B[(int64_t)d * M + min(m, M - 1)]);
  if (bad) s_bad[lane] = 1;
  __syncthreads();
  const uint64_t mask = __ballot(s_bad[lane] != 0);   // (a column past M repeats M - 1; its bit is not read)
  const int words = M - m0 > 32 ? 2 : 1;
  for (int e = tid; e < C * words; e += kWeightThreads)
    reinterpret_cast<uint32_t*>(lut)[(int64_t)(e / words) * kK * M + m0 + e % words] =
        (uint32_t)(mask >> (32 * (e % words)));
}

// a given double table (a fitted one)
struct SrcT {
  const double* T;
  int M;
  __device__ double at(int64_t row, int m) const { return T[row * M + m]; }
  __device__ void at_many(int c, int e0, int stride, int per, double* t) const {
#pragma unroll
    for (int q = 0; q < kStatsILP; ++q) {
      const int e = min(e0 + q * stride, per - 1);
      t[q] = T[(int64_t)c * kK * M + e];
    }
  }
};

template <int NT>
__device__ double block_reduce(double v, bool take_max, double* s_red) {
  const int tid = threadIdx.x;
  s_red[tid] = v;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (tid < w) {
      const double o = s_red[tid + w];
      s_red[tid] = take_max ? fmax(s_red[tid], o) : fmin(s_red[tid], o);
    }
    __syncthreads();
  }
  const double r = s_red[0];
  __syncthreads();
  return r;
}

template <class Src>
__global__ void __launch_bounds__(kStatsThreads)
table_stats_kernel(const Src src, int M, float* __restrict__ scale_out, float* __restrict__ offset_out) {
  __shared__ double s_red[kStatsThreads];
  const int c = blockIdx.x;
  const int per = kK * M;
  double lo = __builtin_inf(), hi = -__builtin_inf();
  for (int e0 = threadIdx.x; e0 < per; e0 += kStatsILP * kStatsThreads) {
    double t[kStatsILP];
    src.at_many(c, e0, kStatsThreads, per, t);
#pragma unroll
    for (int q = 0; q < kStatsILP; ++q)
      if (e0 + q * kStatsThreads < per) {
        lo = fmin(lo, t[q]);
        hi = fmax(hi, t[q]);
      }
  }
  lo = block_reduce<kStatsThreads>(lo, false, s_red);
  hi = block_reduce<kStatsThreads>(hi, true, s_red);
  const float o = (float)__ddiv_rn(__dadd_rn(lo, hi), 2.0);
  double r = 0.0;
  for (int e0 = threadIdx.x; e0 < per; e0 += kStatsILP * kStatsThreads) {
    double t[kStatsILP];
    src.at_many(c, e0, kStatsThreads, per, t);
#pragma unroll
    for (int q = 0; q < kStatsILP; ++q)
      if (e0 + q * kStatsThreads < per) r = fmax(r, fabs(__dsub_rn(t[q], (double)o)));
  }
  r = block_reduce<kStatsThreads>(r, true, s_red);
  if (threadIdx.x == 0) {
    int ex = -126;
    while (ex < 127 && r > 127.0 * __builtin_ldexp(1.0, ex)) ++ex;
    offset_out[c] = o;
    reinterpret_cast<int*>(scale_out)[c] = ex;  // parked exponent, replaced by table_scale_kernel
  }
}

__device__ int max_parked_exponent(const float* __restrict__ scale_out, int C, int* s_max) {
  if (threadIdx.x == 0) *s_max = -126;
  __syncthreads();
  const int* parked = reinterpret_cast<const int*>(scale_out);
  for (int c = threadIdx.x; c < C; c += blockDim.x) atomicMax(s_max, parked_exponent(parked[c]));
  __syncthreads();
  return *s_max;
}

template <class Src>
__global__ void __launch_bounds__(kBuildThreads)
table_codes_kernel(const Src src, int C, int M, int cap, const float* __restrict__ scale_out,
                   const float* __restrict__ offset_out, int8_t* __restrict__ lut) {
  __shared__ int s_max;
  const int emax = max_parked_exponent(scale_out, C, &s_max);
  const int64_t total = (int64_t)C * kK * M;
  for (int64_t e = (int64_t)blockIdx.x * kBuildThreads + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * kBuildThreads) {
    const int64_t row = e / M;
    const int m = (int)(e - row * M);
    const int c = (int)(row / kK);
    const int ex = max(reinterpret_cast<const int*>(scale_out)[c], emax - cap);
    const double t = src.at(row, m);
    const double q = rint(__dmul_rn(__dsub_rn(t, (double)offset_out[c]), __builtin_ldexp(1.0, -ex)));
    lut[e] = (int8_t)(int)fmin(127.0, fmax(-127.0, q));
  }
}

__global__ void table_scale_kernel(float* __restrict__ scale_out, int C, int cap) {
  __shared__ int s_max;
  const int emax = max_parked_exponent(scale_out, C, &s_max);
  // every thread has read its exponents before any is replaced
  int ex[4];
  for (int j = 0; j < 4; ++j) {
    const int c = threadIdx.x + j * blockDim.x;
    ex[j] = c < C ? max(parked_exponent(reinterpret_cast<const int*>(scale_out)[c]), emax - cap) : 0;
  }
  __syncthreads();
  for (int j = 0; j < 4; ++j) {
    const int c = threadIdx.x + j * blockDim.x;
    if (c < C) scale_out[c] = __builtin_ldexpf(1.0f, ex[j]);
  }
}

static unsigned grid_for(int64_t total) {
  const int64_t g = (total + kBuildThreads - 1) / kBuildThreads;
  return (unsigned)(g < 65536 ? (g > 0 ? g : 1) : 65536);
}

template <class Src>
static hipError_t quantize(const Src& src, int C, int M, int8_t* lut, float* scale, float* offset, int cap,
                           hipStream_t stream) {
  hipLaunchKernelGGL(table_stats_kernel<Src>, dim3(C), dim3(kStatsThreads), 0, stream, src, M, scale, offset);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(table_codes_kernel<Src>, dim3(grid_for((int64_t)C * kK * M)), dim3(kBuildThreads), 0,
                     stream, src, C, M, cap, scale, offset, lut);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // C <= 4 * 256 codebooks per single-workgroup scale pass
  hipLaunchKernelGGL(table_scale_kernel, dim3(1), dim3(256), 0, stream, scale, C, cap);
  return hipGetLastError();
}

// The tile.  4 columns per thread (vector loads where the rows of B and of the
// codes are whole 16- and 4-byte units) when that leaves a workgroup for every
// CU, else 1, so that small tables are spread over more of them.  Narrow tables,
// and fp32 ones of few codebooks, are spread over the prototypes too: with 16 of
// them per thread most threads have none of up to 128 columns, and the others
// 16 chains (prototypes without zero columns, 512 codebooks, 10 columns, 16 / 1
// per thread: D 300 364 / 72 us with codes, 170 / 29 fp32; one codebook, D 1024,
// 4096 columns fp32, 16 / 4 per thread, 236 / 94).
template <class F>
static hipError_t with_tile(const void* B, const void* lut, int lut_elem, int C, int D, int M, int cus, F&& f) {
  if (M <= 16) return f(Tile<1, false, 1>{}, 1);
  if (M <= 64) return f(Tile<1, false, 4>{}, 1);
  if (M <= 128) return f(Tile<1, false, 8>{}, 1);
  using Wide = Tile<4, true, kK>;
  using One = Tile<1, false, kK>;
  const int64_t wide = (int64_t)C * ((M + Wide::kCols - 1) / Wide::kCols);
  if (wide < cus) {
    const int ones = (M + One::kCols - 1) / One::kCols;
    if (lut_elem == 4 && D > 16 && 2 * (int64_t)C * ones < cus)
      return f(Tile<1, false, 4>{}, (M + 63) / 64);
    return f(One{}, ones);
  }
  const int tiles = (int)(wide / C);
  const bool vec = M % 4 == 0 && reinterpret_cast<uintptr_t>(B) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(lut) % (4 * lut_elem) == 0;
  if (vec) return f(Wide{}, tiles);
  return f(Tile<4, false, kK>{}, tiles);
}

// Few weights: at most 16 per thread of a tile, which every workgroup looks
// through in less than a launch takes.
template <class T>
static bool few_weights(int D) {
  return (int64_t)D * T::kCols <= 16 * kBuildThreads;
}

hipError_t launch_build_lut(const float* P, const float* B, int C, int D, int M, int8_t* lut,
                            float* scale, float* offset, int cap, int cus, hipStream_t stream) {
  hipError_t e = with_tile(B, lut, 1, C, D, M, cus, [&](auto tile, int tiles) {
    using T = decltype(tile);
    const dim3 grid((unsigned)(C * tiles)), block(kBuildThreads);
    hipError_t r;
    if (tiles == 1 && few_weights<T>(D)) {
      hipLaunchKernelGGL(build_small_exponent_kernel<T>, dim3(C), block, 0, stream, P, B, D, M, scale, offset);
    } else {
      hipLaunchKernelGGL(build_range_kernel<T>, grid, block, 0, stream, P, B, C, D, M, tiles, lut);
      if ((r = hipGetLastError()) != hipSuccess) return r;
      hipLaunchKernelGGL(build_exponent_kernel<T>, dim3(C), block, 0, stream, P, B, C, D, M, tiles, lut, scale, offset);
    }
    if ((r = hipGetLastError()) != hipSuccess) return r;
    hipLaunchKernelGGL(build_codes_kernel<T>, grid, block, 0, stream, P, B, C, D, M, tiles, cap, scale, offset, lut);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  // C <= 4 * 256 codebooks per single-workgroup scale pass
  hipLaunchKernelGGL(table_scale_kernel, dim3(1), dim3(256), 0, stream, scale, C, cap);
  return hipGetLastError();
}

hipError_t launch_quantize_lut(const double* T, int C, int M, int8_t* lut, float* scale, float* offset, int cap,
                               hipStream_t stream) {
  return quantize(SrcT{T, M}, C, M, lut, scale, offset, cap, stream);
}

hipError_t launch_build_lut_f32(const float* P, const float* B, int C, int D, int M, float* lut, int cus,
                                hipStream_t stream) {
  // Up to 16 columns of P and a few million products: an entry per thread (D 16,
  // an entry per thread / in tiles: 16 x 256 3.7 / 6.5 us, 128 x 1000 13 / 7).
  if (D <= 16 && (int64_t)C * kK * M * D <= 6000000) {
    const int total = C * kK * M;
    hipLaunchKernelGGL(build_f32_small_kernel, dim3(grid_for(total)), dim3(kBuildThreads), 0, stream, P, B, D, M, total,
                       lut);
    return hipGetLastError();
  }
  return with_tile(B, lut, 4, C, D, M, cus, [&](auto tile, int tiles) {
    using T = decltype(tile);
    const dim3 grid((unsigned)(C * tiles)), block(kBuildThreads);
    if (few_weights<T>(D)) {
      hipLaunchKernelGGL((build_f32_kernel<T, true>), grid, block, 0, stream, P, B, C, D, M, tiles, lut);
      return hipGetLastError();
    }
    hipLaunchKernelGGL(weights_kernel, dim3((unsigned)((M + 63) / 64)), dim3(kWeightThreads), 0, stream, B, C, D, M, lut);
    hipError_t r = hipGetLastError();
    if (r != hipSuccess) return r;
    hipLaunchKernelGGL((build_f32_kernel<T, false>), grid, block, 0, stream, P, B, C, D, M, tiles, lut);
    return hipGetLastError();
  });
}

}  // namespace mdn
