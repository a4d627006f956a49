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
// exponent (parked in scale_out as an integer); the codes; the scales.  The
// entries are evaluated in the first and the third (no workspace for a double
// copy of T).  A given table T takes three: statistics (one workgroup per
// codebook), codes, scales.
//
// Zero prototype columns.  P[c] is zero outside codebook c's subspace, so most
// terms are a zero times a finite weight.  A sum that starts at +0 is never
// -0 and adding +-0 to it changes nothing, so a column d with P[c][k][d] = 0
// for all 16 k is skipped with the sum's bits unchanged, as long as every
// B[d][m] is finite (0 * inf and 0 * NaN are NaN).  Each workgroup lists the
// columns of its codebook that are not all zero, ascending, and the weights
// are checked on the way: every (codebook, tile) checks its share of B's rows.
// One non-finite weight anywhere, and every column is taken.
//
// Bound: launches and latency (P and B once from HBM, a few columns per
// codebook); with prototypes that have no zero column, the fp64 FMA rate.
// 128 codebooks, D 1024, M 4096 (8 nonzero columns per codebook): 57 us a build
// against 14.2 ms with every column taken and one workgroup per codebook.
#include "internal.hpp"

namespace mdn {

constexpr int kBuildThreads = 256;
// the statistics pass: one workgroup of kStatsThreads per codebook, kStatsILP
// entries of a thread evaluated together (their sums are independent chains,
// each in its own order)
constexpr int kStatsThreads = 1024;
constexpr int kStatsILP = 4;

constexpr int kChunk = 512;   // prototype columns listed at a time

// What a workgroup of kBuildThreads keeps of one chunk of P[c]: the columns
// that are not all zero, ascending, and their 16 values (as doubles: they are
// read once per column of the tile).
struct TileLds {
  double p[kChunk][kK];
  int d[kChunk];
  int cnt[2 * kBuildThreads / 64];
};

// The 16 x (CPT kBuildThreads) tile of T from column col0 of codebook c: this
// thread's columns are colof(j), t[k][j] their sums over d ascending.  The
// product of two floats is exact in double, so the fused multiply-add rounds
// exactly as a multiply and an add do.  `dense` takes the zero columns too.
// Columns past M read column M - 1.
template <int CPT, bool VEC>
struct Tile {
  static constexpr int kCpt = CPT;
  static constexpr bool kVec = VEC;
  static constexpr int kCols = CPT * kBuildThreads;
  static __device__ __forceinline__ int colof(int col0, int j) {
    return VEC ? col0 + CPT * (int)threadIdx.x + j : col0 + (int)threadIdx.x + j * kBuildThreads;
  }
  static __device__ void sums(const float* __restrict__ P, const float* __restrict__ B, int D, int M, int c, int col0,
                              bool dense, TileLds& s, double (&t)[kK][CPT]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NW = kBuildThreads / 64;
#pragma unroll
    for (int k = 0; k < kK; ++k)
#pragma unroll
      for (int j = 0; j < CPT; ++j) t[k][j] = 0.0;
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
      __syncthreads();   // the previous chunk's (or tile's) list has been read
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
      constexpr int kU = 4;   // rows of B in flight
      for (int e0 = 0; e0 < n; e0 += kU) {
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
            for (int k = 0; k < kK; ++k) {
              const double pv = s.p[e0 + u][k];
#pragma unroll
              for (int j = 0; j < CPT; ++j) t[k][j] = __fma_rn(pv, (double)w[u][j], t[k][j]);
            }
          }
      }
    }
  }
};

// a double at any byte address (the codes are a byte array)
struct __attribute__((packed)) F64u { double v; };

// The range of T over one (codebook, column tile), parked in the first 16
// bytes of the tile's codes ([lo, hi]; a tile of any codebook has at least 16
// bytes).  lo = NaN says that a weight among this workgroup's share of B is
// not finite (a range of entries is never NaN: fmin and fmax skip NaN).
template <int CPT, bool VEC>
__global__ void __launch_bounds__(kBuildThreads)
build_range_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M, int tiles,
                   int8_t* lut) {
  __shared__ TileLds s;
  __shared__ double s_red[2][kBuildThreads / 64];
  __shared__ int s_bad;
  using T = Tile<CPT, VEC>;
  const int c = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const int col0 = tile * T::kCols;
  if (threadIdx.x == 0) s_bad = 0;
  double t[kK][CPT];
  T::sums(P, B, D, M, c, col0, false, s, t);   // (has barriers: s_bad is set)
  bool bad = false;
  for (int d = (int)((int64_t)c * D / C); d < (int)((int64_t)(c + 1) * D / C); ++d)
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      bad |= !__builtin_isfinite(B[(int64_t)d * M + min(T::colof(col0, j), M - 1)]);
  if (bad) s_bad = 1;
  double lo = __builtin_inf(), hi = -__builtin_inf();
#pragma unroll
  for (int j = 0; j < CPT; ++j)
    if (T::colof(col0, j) < M)
#pragma unroll
      for (int k = 0; k < kK; ++k) {
        lo = fmin(lo, t[k][j]);
        hi = fmax(hi, t[k][j]);
      }
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o));
    hi = fmax(hi, __shfl_xor(hi, o));
  }
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = lo;
    s_red[1][threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBuildThreads / 64; ++w) {
      lo = fmin(lo, s_red[0][w]);
      hi = fmax(hi, s_red[1][w]);
    }
    F64u* out = reinterpret_cast<F64u*>(lut + (int64_t)c * kK * M + 16 * tile);
    out[0].v = s_bad ? __builtin_nan("") : lo;
    out[1].v = hi;
  }
}

constexpr int kDenseBit = 1 << 16;   // in a parked exponent: take every prototype column

// Offset and exponent of codebook c = blockIdx.x from its tiles' ranges.
// r = max |T - o| is taken at an end of the range (rounding is monotone).
// With a non-finite weight anywhere the range is evaluated here over every
// prototype column, and the codes are told to do the same.
template <int CPT, bool VEC>
__global__ void __launch_bounds__(kBuildThreads)
build_exponent_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M, int tiles,
                      const int8_t* lut, float* __restrict__ scale_out, float* __restrict__ offset_out) {
  __shared__ TileLds s;
  __shared__ double s_red[2][kBuildThreads / 64];
  __shared__ int s_bad;
  using T = Tile<CPT, VEC>;
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
      double t[kK][CPT];
      T::sums(P, B, D, M, c, tile * T::kCols, true, s, t);
#pragma unroll
      for (int j = 0; j < CPT; ++j)
        if (T::colof(tile * T::kCols, j) < M)
#pragma unroll
          for (int k = 0; k < kK; ++k) {
            lo = fmin(lo, t[k][j]);
            hi = fmax(hi, t[k][j]);
          }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o));
    hi = fmax(hi, __shfl_xor(hi, o));
  }
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = lo;
    s_red[1][threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBuildThreads / 64; ++w) {
      lo = fmin(lo, s_red[0][w]);
      hi = fmax(hi, s_red[1][w]);
    }
    const float o = (float)__ddiv_rn(__dadd_rn(lo, hi), 2.0);
    const double r = fmax(fmax(0.0, fabs(__dsub_rn(lo, (double)o))), fabs(__dsub_rn(hi, (double)o)));
    int ex = -126;
    while (ex < 127 && r > 127.0 * __builtin_ldexp(1.0, ex)) ++ex;
    offset_out[c] = o;
    // parked, replaced by table_scale_kernel
    reinterpret_cast<int*>(scale_out)[c] = ex + (dense ? kDenseBit : 0);
  }
}

__device__ __forceinline__ int parked_exponent(int v) { return v >= kDenseBit / 2 ? v - kDenseBit : v; }

__device__ __forceinline__ int8_t code_of(double t, double o, double inv) {
  return (int8_t)(int)fmin(127.0, fmax(-127.0, rint(__dmul_rn(__dsub_rn(t, o), inv))));
}

__device__ int max_parked_exponent(const float* __restrict__ scale_out, int C, int* s_max);

template <int CPT, bool VEC>
__global__ void __launch_bounds__(kBuildThreads)
build_codes_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M, int tiles, int cap,
                   const float* __restrict__ scale_out, const float* __restrict__ offset_out,
                   int8_t* __restrict__ lut) {
  __shared__ TileLds s;
  __shared__ int s_max;
  using T = Tile<CPT, VEC>;
  const int c = blockIdx.x / tiles, col0 = (blockIdx.x % tiles) * T::kCols;
  const int parked = reinterpret_cast<const int*>(scale_out)[c];
  double t[kK][CPT];
  T::sums(P, B, D, M, c, col0, parked >= kDenseBit / 2, s, t);
  const int ex = max(parked_exponent(parked), max_parked_exponent(scale_out, C, &s_max) - cap);
  const double o = (double)offset_out[c], inv = __builtin_ldexp(1.0, -ex);
  int8_t* out = lut + (int64_t)c * kK * M;
#pragma unroll
  for (int k = 0; k < kK; ++k) {
    if constexpr (VEC) {   // M % 4 == 0: a thread's 4 columns exist together
      const int m = T::colof(col0, 0);
      if (m < M) {
        uint32_t q = 0;
#pragma unroll
        for (int j = 0; j < CPT; ++j) q |= (uint32_t)(uint8_t)code_of(t[k][j], o, inv) << (8 * j);
        *reinterpret_cast<uint32_t*>(out + (int64_t)k * M + m) = q;
      }
    } else {
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const int m = T::colof(col0, j);
        if (m < M) out[(int64_t)k * M + m] = code_of(t[k][j], o, inv);
      }
    }
  }
}

template <int CPT, bool VEC>
__global__ void __launch_bounds__(kBuildThreads)
build_f32_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M, int tiles,
                 float* __restrict__ lut) {
  __shared__ TileLds s;
  using T = Tile<CPT, VEC>;
  const int c = blockIdx.x / tiles, col0 = (blockIdx.x % tiles) * T::kCols;
  double t[kK][CPT];
  T::sums(P, B, D, M, c, col0, false, s, t);
  float* out = lut + (int64_t)c * kK * M;
#pragma unroll
  for (int k = 0; k < kK; ++k) {
    if constexpr (VEC) {
      const int m = T::colof(col0, 0);
      if (m < M)
        *reinterpret_cast<float4*>(out + (int64_t)k * M + m) =
            make_float4((float)t[k][0], (float)t[k][1], (float)t[k][2], (float)t[k][3]);
    } else {
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const int m = T::colof(col0, j);
        if (m < M) out[(int64_t)k * M + m] = (float)t[k][j];
      }
    }
  }
}

// The fp32 table's entries of columns that hold a non-finite weight, over
// every prototype column (the launch above skipped the zero ones): 64 columns
// per workgroup, which reads them through once and is done if all are finite.
constexpr int kRepairThreads = 1024;
__global__ void __launch_bounds__(kRepairThreads)
build_f32_repair_kernel(const float* __restrict__ P, const float* __restrict__ B, int C, int D, int M,
                        float* __restrict__ lut) {
  __shared__ int s_bad[64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int m = blockIdx.x * 64 + lane;
  if (tid < 64) s_bad[tid] = 0;
  __syncthreads();
  bool bad = false;
#pragma unroll 8
  for (int d = tid >> 6; d < D; d += kRepairThreads / 64)
    bad |= !__builtin_isfinite(B[(int64_t)d * M + min(m, M - 1)]);
  if (bad && m < M) s_bad[lane] = 1;
  __syncthreads();
  if (m >= M || !s_bad[lane]) return;
  for (int row = tid >> 6; row < C * kK; row += kRepairThreads / 64) {
    double t = 0.0;
    for (int d = 0; d < D; ++d)
      t = __fma_rn((double)P[(int64_t)row * D + d], (double)B[(int64_t)d * M + m], t);
    lut[(int64_t)row * M + m] = (float)t;
  }
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

// Columns per thread of a tile: 4 (vector loads where the rows of B and of the
// codes are whole 16- and 4-byte units) when that leaves a workgroup for every
// CU, else 1, so that small tables are spread over more of them.
template <class F>
static hipError_t with_tile(const void* B, const void* lut, int lut_elem, int C, int M, int cus, F&& f) {
  const int64_t wide = (int64_t)C * ((M + Tile<4, true>::kCols - 1) / Tile<4, true>::kCols);
  if (wide < cus) return f(Tile<1, false>{}, (M + Tile<1, false>::kCols - 1) / Tile<1, false>::kCols);
  const int tiles = (int)(wide / C);
  const bool vec = M % 4 == 0 && reinterpret_cast<uintptr_t>(B) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(lut) % (4 * lut_elem) == 0;
  if (vec) return f(Tile<4, true>{}, tiles);
  return f(Tile<4, false>{}, tiles);
}

hipError_t launch_build_lut(const float* P, const float* B, int C, int D, int M, int8_t* lut,
                            float* scale, float* offset, int cap, int cus, hipStream_t stream) {
  hipError_t e = with_tile(B, lut, 1, C, M, cus, [&](auto tile, int tiles) {
    constexpr int CPT = decltype(tile)::kCpt;
    constexpr bool VEC = decltype(tile)::kVec;
    const dim3 grid((unsigned)(C * tiles)), block(kBuildThreads);
    hipLaunchKernelGGL((build_range_kernel<CPT, VEC>), grid, block, 0, stream, P, B, C, D, M, tiles, lut);
    hipError_t r = hipGetLastError();
    if (r != hipSuccess) return r;
    hipLaunchKernelGGL((build_exponent_kernel<CPT, VEC>), dim3(C), block, 0, stream, P, B, C, D, M, tiles, lut, scale,
                       offset);
    if ((r = hipGetLastError()) != hipSuccess) return r;
    hipLaunchKernelGGL((build_codes_kernel<CPT, VEC>), grid, block, 0, stream, P, B, C, D, M, tiles, cap, scale,
                       offset, lut);
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
  hipError_t e = with_tile(B, lut, 4, C, M, cus, [&](auto tile, int tiles) {
    hipLaunchKernelGGL((build_f32_kernel<decltype(tile)::kCpt, decltype(tile)::kVec>), dim3((unsigned)(C * tiles)),
                       dim3(kBuildThreads), 0, stream, P, B, C, D, M, tiles, lut);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(build_f32_repair_kernel, dim3((unsigned)((M + 63) / 64)), dim3(kRepairThreads), 0, stream, P, B,
                     C, D, M, lut);
  return hipGetLastError();
}

}  // namespace mdn
