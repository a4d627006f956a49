// Model-aware table fit, Eq. 3 of McCarter & Dronen (§2.2), with an affine
// layer output (bias and identity, which cancel): the table T minimising
// ||Y - G T||^2 + lambda ||T - T0||^2 solves the normal equations
//     (G^T G + lambda I) T = G^T Y + lambda T0,
// G the one-hot encoder output (G[n][16c + k] = 1 iff idx[n][c] = k), Y = AB
// the layer's exact outputs on training rows and T0 = P0 B the prototype
// table.  Offline: it turns training data into a table for the hot path.
//
// Steps (each its own launch family):
//   gram    H = G^T G, integer counts: H[16c + k][16c' + k'] is the number of
//           rows whose codebook-c index is k and codebook-c' index is k'.
//           Workgroups own an 8 x 8 block of codebook pairs and a row chunk,
//           count in LDS, then add their nonzero counts to H (integer
//           atomics: the result does not depend on their order).
//   scatter R = G^T Y in double: a stable counting sort lists each
//           codebook's rows bucket by bucket (ascending within a bucket),
//           then one workgroup per (codebook, bucket, 64 columns)
//           sums the bucket's rows in that order: every entry is the
//           sum of its rows in ascending row order.
//   solve   A = H + lambda I (double), B = R + lambda T0; A = L L^T by a
//           blocked right-looking Cholesky factorisation (panels of 32: the
//           panel, then the trailing update), then blocked forward and
//           backward substitution over the M columns of B, in place.
// Every multiply-subtract is one fused multiply-add, and every entry takes
// its terms in the same order as the unblocked algorithm (k ascending in the
// factor and forward pass, descending in the backward pass), so the result
// does not depend on the blocking.
#include "internal.hpp"

namespace mdn {

namespace {

constexpr int kNB = 32;        // panel / block width of the factorisation and the solves
constexpr int kGB = 8;         // codebooks per side of a Gram pair block
constexpr int kGW = kGB * kK;  // 128: counts per side of a pair block

__global__ void __launch_bounds__(256) fill_i32_kernel(int32_t* __restrict__ p, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) p[e] = 0;
}

// ------------------------------------------------------------------ gram
__global__ void __launch_bounds__(256)
gram_kernel(const uint8_t* __restrict__ idx, int64_t N, int C, int nbc, int64_t chunk_rows,
            int32_t* __restrict__ H) {
  __shared__ int s_cnt[kGW * kGW];   // 64 KB
  const int tid = threadIdx.x;
  const int npair = nbc * nbc;
  const int pair = blockIdx.x % npair;
  const int64_t chunk = blockIdx.x / npair;
  const int c1 = (pair / nbc) * kGB, c2 = (pair % nbc) * kGB;
  const int n1 = min(kGB, C - c1), n2 = min(kGB, C - c2);
  for (int e = tid; e < kGW * kGW; e += 256) s_cnt[e] = 0;
  __syncthreads();
  const int64_t r0 = chunk * chunk_rows;
  const int64_t r1 = min(N, r0 + chunk_rows);
  for (int64_t n = r0 + tid; n < r1; n += 256) {
    const uint8_t* ir = idx + n * C;
    int ka[kGB], kb[kGB];
#pragma unroll
    for (int a = 0; a < kGB; ++a) ka[a] = a < n1 ? (int)(ir[c1 + a] & 15) : 0;
#pragma unroll
    for (int b = 0; b < kGB; ++b) kb[b] = b < n2 ? (int)(ir[c2 + b] & 15) : 0;
#pragma unroll
    for (int a = 0; a < kGB; ++a)
#pragma unroll
      for (int b = 0; b < kGB; ++b)
        if (a < n1 && b < n2) atomicAdd(&s_cnt[(a * kK + ka[a]) * kGW + b * kK + kb[b]], 1);
  }
  __syncthreads();
  const int64_t n16 = (int64_t)C * kK;
  for (int e = tid; e < kGW * kGW; e += 256) {
    const int v = s_cnt[e];
    const int ra = e / kGW, rb = e % kGW;
    if (v != 0 && ra < n1 * kK && rb < n2 * kK) atomicAdd(&H[(c1 * kK + ra) * n16 + c2 * kK + rb], v);
  }
}

// --------------------------------------------------------------- scatter
// R[16c + k][m] = sum over rows n (ascending) with idx[n][c] = k of Y[n][m].
//
// partition: one workgroup per codebook lists the rows bucket by bucket,
// ascending within each bucket (a stable counting sort), perm[c][start_k ..] =
// rows of bucket k, start[c][k] the bucket starts (start[c][16] = N).
// The lists lie N + 128 entries apart, so that a power of two of rows does not put
// them at the same distance from each other's memory channels and cache sets (ten
// gradient steps on 16,384 rows, 32 x 64: 1256 us, 1282 packed).  Nothing is kept
// in the gaps.
constexpr int kListGap = 128;

constexpr int kPartWaves = 16;

// One workgroup per codebook; wavefront w takes the w-th contiguous run of
// whole 64-row batches, counts its buckets, and after one barrier knows where
// its rows of each bucket go (bucket-major, then wavefront: stable).  The
// rank of a row among its batch's rows of the same bucket comes from 4 ballots
// (one per index bit).  Bound: load latency, 8 batches requested together
// (16,384 rows x 64 codebooks: 312 -> 23 us against one
// wavefront per codebook).
__global__ void __launch_bounds__(kPartWaves * 64)
partition_kernel(const uint8_t* __restrict__ idx, int64_t N, int C, int32_t* __restrict__ perm,
                 int32_t* __restrict__ start) {
  __shared__ int s_cnt[kPartWaves][kK];   // rows per bucket of a wavefront, then its next position
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = blockIdx.x;
  const uint64_t lt = (1ull << lane) - 1;   // lanes below this one
  const int64_t batches = (N + 63) / 64;
  const int64_t b0 = batches * wave / kPartWaves, b1 = batches * (wave + 1) / kPartWaves;
  constexpr int kU = 8;
  auto load = [&](int64_t b, int (&key)[kU]) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t n = (b + u) * 64 + lane;
      key[u] = b + u < b1 && n < N ? (int)(idx[n * C + c] & 15) : kK;
    }
  };
  // lanes of this batch whose row is in the same bucket (key < 16)
  auto same = [&](int key) {
    uint64_t m = __ballot(key < kK);
#pragma unroll
    for (int bit = 0; bit < 4; ++bit) {
      const uint64_t v = __ballot((key >> bit) & 1);
      m &= (key >> bit) & 1 ? v : ~v;
    }
    return m;
  };
  // orders a wavefront's own LDS accesses across its lanes (no instruction)
  auto in_order = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (lane < kK) s_cnt[wave][lane] = 0;
  in_order();
  for (int64_t b = b0; b < b1; b += kU) {
    int key[kU];
    load(b, key);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint64_t m = same(key[u]);
      if (key[u] < kK && (m & lt) == 0) s_cnt[wave][key[u]] += __popcll(m);
      in_order();
    }
  }
  __syncthreads();
  if (threadIdx.x < kK) {   // lane k: the bucket's rows in all, the buckets before it, then its wavefronts
    int total = 0;
    for (int w = 0; w < kPartWaves; ++w) total += s_cnt[w][lane];
    int run = total;
    for (int o = 1; o < kK; o <<= 1) {
      const int v = __shfl_up(run, o);
      if (lane >= o) run += v;
    }
    run -= total;
    start[c * (kK + 1) + lane] = run;
    for (int w = 0; w < kPartWaves; ++w) {
      const int v = s_cnt[w][lane];
      s_cnt[w][lane] = run;
      run += v;
    }
  }
  if (threadIdx.x == 0) start[c * (kK + 1) + kK] = (int32_t)N;
  __syncthreads();
  int32_t* pc = perm + (int64_t)c * (N + kListGap);
  for (int64_t b = b0; b < b1; b += kU) {
    int key[kU];
    load(b, key);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint64_t m = same(key[u]);
      const int at = s_cnt[wave][key[u] & 15];
      in_order();
      if (key[u] < kK) {
        pc[at + __popcll(m & lt)] = (int32_t)((b + u) * 64 + lane);
        if ((m & lt) == 0) s_cnt[wave][key[u]] = at + __popcll(m);
      }
      in_order();
    }
  }
}

// scatter: one workgroup per (codebook, bucket, TC columns) walks the bucket's
// rows in stages.  Seven wavefronts load them (8 rows per lane and stage,
// 64 / TC row groups side by side, some stages ahead in registers) and hand
// them over through LDS, 16 bytes per lane and access (2 rows of doubles or 4
// of floats of one column together); the first wavefront, lane = column, adds
// them: every entry is its bucket's rows summed in ascending order.  V: float
// (targets Y) or double (gradient residuals).  `done(bucket row, column, sum)`
// takes the result: stores it, or takes the gradient step.
//
// The sum of a bucket is one chain of dependent adds, and buckets are uneven
// (the largest of a random tree's 16 holds about half of the rows), so the adding
// wavefront does nothing else.  Bound: on small layers that wavefront, at about 20
// cycles a row with its LDS reads and its loop (of the 81 us below, 76 are left
// without the loads from memory, 38 without the adds), on large ones the L2 as
// well, which reads every row once per codebook.  Column tiles go to XCDs
// (workgroup b runs on XCD b % 8): with a
// number of tiles that divides 8, or a multiple of 8, each XCD reads its own
// columns only, and TC is such that they fit its 4 MB L2 at the training sets'
// sizes; else the tiles are taken one after the other.
// Measured against one wavefront per codebook with its 16 buckets in turn:
// 16,384 rows, 32 codebooks x 64 columns of doubles 554 -> 81 us (largest
// bucket 9063 rows); 64 codebooks x 512 columns of floats 585 -> 163 us (2.1 GB
// out of the L2s).
constexpr int kScWaves = 8, kScPer = 8;   // wavefronts; rows of a loading lane per stage

// a barrier that orders LDS only: global loads stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <class V, int TC, class F>
__device__ __forceinline__ void scatter_bucket(const int32_t* __restrict__ perm, const int32_t* __restrict__ start,
                                               int64_t N, int C, const V* __restrict__ Y, int M, F&& done) {
  constexpr int R = 16 / (int)sizeof(V);              // rows of one LDS access
  typedef V Pack __attribute__((ext_vector_type(R)));
  constexpr int kPer = kScPer * (64 / TC);            // rows of a loading wavefront per stage
  constexpr int kRows = (kScWaves - 1) * kPer;        // rows of a stage
  constexpr int kPacks = kRows / R;
  constexpr int kDepth = 64 / kPer < 4 ? 64 / kPer : 4;   // stages in flight; at most one row number per lane
  constexpr int kAhead = 7;                           // LDS reads ahead of the adds
  static_assert(kPacks % kAhead == 0, "whole chunks");
  __shared__ Pack s_row[2][kPacks][TC];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ntile = (M + TC - 1) / TC, rows = C * kK;
  int tile, r;
  if (ntile % 8 == 0) {
    const int j = blockIdx.x >> 3;
    tile = (blockIdx.x & 7) + 8 * (j / rows);
    r = j % rows;
  } else if (8 % ntile == 0) {
    tile = blockIdx.x % ntile;
    r = blockIdx.x / ntile;
  } else {
    tile = blockIdx.x / rows;
    r = blockIdx.x % rows;
  }
  // every codebook's largest bucket first, then the second largest, ...: the
  // long chains start at once
  const int c = r % C;
  int k;
  {
    const int32_t* sc = start + c * (kK + 1);
    const int size = lane < kK ? sc[lane + 1] - sc[lane] : -1;
    int rank = 0;
#pragma unroll
    for (int j = 0; j < kK; ++j) {
      const int o = __builtin_amdgcn_readlane(size, j);
      rank += o > size || (o == size && j < lane);
    }
    k = __ffsll(__ballot(lane < kK && rank == r / C)) - 1;
  }
  const int m = tile * TC + lane % TC;
  const int64_t p0 = start[c * (kK + 1) + k], p1 = start[c * (kK + 1) + k + 1];
  // whole groups of kDepth stages (the last ones may have no rows): no branch
  // in the loaders' loop, where the compiler would wait for every load in
  // flight at the join
  const int64_t nst = (p1 - p0 + kRows * kDepth - 1) / (kRows * kDepth) * kDepth;
  if (wave != 0) {
    // a lane holds one row number of the next kDepth stages (row lane % kPer
    // of stage lane / kPer), read a group of stages ahead; rows past the
    // bucket are its last one, columns past M column M - 1: every load is
    // valid, what is not used is ignored
    if (nst == 0) return;
    const V* yc = Y + min(m, M - 1);
    const int32_t* pc = perm + (int64_t)c * (N + kListGap);
    const int64_t mine = p0 + lane / kPer % kDepth * kRows + (wave - 1) * kPer + lane % kPer;
    const int first = lane / TC * kScPer;   // this lane's first row of the wavefront's
    auto fetch = [&](int64_t st) { return pc[min(mine + st * kRows, p1 - 1)]; };
    V v[kDepth][kScPer];
    auto load = [&](int d, int numbers, V (&to)[kScPer]) {
#pragma unroll
      for (int j = 0; j < kScPer; ++j) {
        const int n = TC == 64 ? __builtin_amdgcn_readlane(numbers, d * kPer + j)
                               : __shfl(numbers, d * kPer + first + j);
        to[j] = yc[(int64_t)n * M];
      }
    };
    auto put = [&](int64_t st, const V (&from)[kScPer]) {
#pragma unroll
      for (int j = 0; j < kScPer; j += R) {
        Pack q;
#pragma unroll
        for (int i = 0; i < R; ++i) q[i] = from[j + i];
        s_row[st & 1][((wave - 1) * kPer + first + j) / R][lane % TC] = q;
      }
    };
    int now = fetch(0), next = fetch(kDepth);
#pragma unroll
    for (int d = 0; d < kDepth; ++d) load(d, now, v[d]);
    put(0, v[0]);
    lds_barrier();
    for (int64_t st = 0; st < nst; st += kDepth) {
      now = next;
      next = fetch(st + 2 * kDepth);
#pragma unroll
      for (int d = 0; d < kDepth; ++d) {   // stage st + d + 1 to LDS, st + d + kDepth requested
        load(d, now, v[d]);
        put(st + d + 1, v[(d + 1) % kDepth]);
        lds_barrier();
      }
    }
    return;
  }
  double acc = 0.0;
  __builtin_amdgcn_s_setprio(3);
  if (nst > 0) lds_barrier();
  for (int64_t st = 0; st < nst; ++st) {
    const Pack(&row)[kPacks][TC] = s_row[st & 1];
    const int64_t left = p1 - p0 - st * kRows;
    // chunks of kAhead packs: the next chunk's reads go out between this one's
    // adds (scheduling barriers: left alone the compiler reads two rows ahead,
    // and reads in groups hold up the adds behind them).  Kept a short loop:
    // unrolled over the stage, most of the time went into fetching its code.
    const int n = (int)(left < kRows ? (left > 0 ? left : 0) : kRows);
    Pack g[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) g[i] = row[i][lane % TC];
    int at = 0;   // first pack of the chunk
#pragma unroll 1
    for (; (at + kAhead) * R <= n; at += kAhead) {
      const int next = at + kAhead < kPacks ? at + kAhead : 0;
#pragma unroll
      for (int i = 0; i < kAhead; ++i) {
#pragma unroll
        for (int j = 0; j < R; ++j) acc = __dadd_rn(acc, (double)g[i][j]);
        g[i] = row[next + i][lane % TC];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the bucket's last rows; those past it add +0: the sum starts at +0 and
    // is never -0
    if (at * R < n) {
#pragma unroll
      for (int i = 0; i < kAhead; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j) acc = __dadd_rn(acc, (at + i) * R + j < n ? (double)g[i][j] : 0.0);
    }
    lds_barrier();
  }
  if (lane < TC && m < M) done((int64_t)c * kK + k, m, acc);
}

// The same sums for small buckets, a wavefront per (codebook, bucket, 64
// columns): 16 rows' loads together, no LDS, so that many buckets are in flight
// where a workgroup each would spend its time on starting and ending.
constexpr int kFewWaves = 4;
template <class V, class F>
__device__ __forceinline__ void scatter_few_rows(const int32_t* __restrict__ perm, const int32_t* __restrict__ start,
                                                 int64_t N, int C, const V* __restrict__ Y, int M, F&& done) {
  constexpr int kU = 16;
  const int lane = threadIdx.x & 63;
  const int ntile = (M + 63) / 64;
  const int64_t w = (int64_t)blockIdx.x * kFewWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (w >= (int64_t)C * kK * ntile) return;   // uniform
  const int64_t r = w / ntile;   // bucket 16 c + k
  const int c = (int)(r / kK), k = (int)(r % kK);
  const int m = (int)(w % ntile) * 64 + lane;
  const V* yc = Y + min(m, M - 1);   // columns past M read column M - 1
  const int32_t* pc = perm + (int64_t)c * (N + kListGap);
  const int64_t p0 = start[c * (kK + 1) + k], p1 = start[c * (kK + 1) + k + 1];
  double acc = 0.0;
  for (int64_t p = p0; p < p1; p += 64) {
    const int cnt = (int)min((int64_t)64, p1 - p);
    const int numbers = pc[min(p + lane, p1 - 1)];   // one row number per lane
    for (int j = 0; j < cnt; j += kU) {
      V v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u)
        v[u] = yc[(int64_t)__builtin_amdgcn_readlane(numbers, min(j + u, cnt - 1)) * M];
      // (rows past the bucket add +0: the sum starts at +0 and is never -0)
#pragma unroll
      for (int u = 0; u < kU; ++u) acc = __dadd_rn(acc, j + u < cnt ? (double)v[u] : 0.0);
    }
  }
  if (m < M) done(r, m, acc);
}

constexpr int kScCols = 64;                                            // columns of floats per workgroup
// of doubles: at most 8 tiles of 16 for narrow layers (their chains are what
// counts: 79 us against 86 with 32 columns, C 32, M 64), else 64 (the LDS is what
// counts, and narrower tiles leave most of an access unused: C 256, M 1024 2.8 ms
// a step against 6.9 with 32 columns).  No width of 65 to 512 columns, with 1 to
// 256 codebooks and 2000 to 65,536 rows, is slower than with a wavefront per
// codebook.
constexpr int step_cols(int M) { return M <= 128 ? 16 : 64; }
unsigned scatter_grid(int C, int M, int cols) { return (unsigned)(C * kK * ((M + cols - 1) / cols)); }
unsigned few_rows_grid(int C, int M) {
  return (unsigned)(((int64_t)C * kK * ((M + 63) / 64) + kFewWaves - 1) / kFewWaves);
}
// Where a wavefront per bucket is the faster one, also when one bucket holds
// half of the rows (us, with random trees' buckets, a workgroup / a wavefront
// each): the sums 64 codebooks x 512 columns 53 / 31 at 500 rows, 56 / 52 at 1000,
// 61 / 96 at 2000, 256 x 1024 347 / 104, 370 / 185; three gradient steps of 256
// x 128 916 / 219 at 500 rows, 1028 / 501 at 2000, 1305 / 930 at 4096, of 128 x
// 10 111 / 83, 121 / 145, 150 / 247, and of 128 x 512 1011 / 545, 1093 / 1202.
bool few_rows_sum(int64_t N, int C, int M) { return N <= 1024 && scatter_grid(C, M, kScCols) >= 8 * N; }
bool few_rows_step(int64_t N, int C, int M) {
  return N <= (step_cols(M) == 16 ? 8192 : 1024) && scatter_grid(C, M, step_cols(M)) >= 4 * N;
}

__global__ void __launch_bounds__(kScWaves * 64)
scatter_kernel(const int32_t* __restrict__ perm, const int32_t* __restrict__ start, int64_t N, int C,
               const float* __restrict__ Y, int M, double* __restrict__ R) {
  scatter_bucket<float, kScCols>(perm, start, N, C, Y, M, [&](int64_t r, int m, double v) { R[r * M + m] = v; });
}
__global__ void __launch_bounds__(kFewWaves * 64)
scatter_few_kernel(const int32_t* __restrict__ perm, const int32_t* __restrict__ start, int64_t N, int C,
                   const float* __restrict__ Y, int M, double* __restrict__ R) {
  scatter_few_rows<float>(perm, start, N, C, Y, M, [&](int64_t r, int m, double v) { R[r * M + m] = v; });
}

// The gradient step on the sums just made: T = T - eta (R + 2 lambda (T - T0))
struct GradStep {
  const float* T0;
  double two_lam, eta;
  double* T;
  int M;
  __device__ void operator()(int64_t r, int m, double v) const {
    const int64_t e = r * M + m;
    const double g = __dadd_rn(v, __dmul_rn(two_lam, __dsub_rn(T[e], (double)T0[e])));
    T[e] = __dsub_rn(T[e], __dmul_rn(eta, g));
  }
};
template <int TC>
__global__ void __launch_bounds__(kScWaves * 64)
scatter_step_kernel(const int32_t* __restrict__ perm, const int32_t* __restrict__ start, int64_t N, int C,
                    const double* __restrict__ Dv, int M, const float* __restrict__ T0, double lam, double eta,
                    double* __restrict__ T) {
  scatter_bucket<double, TC>(perm, start, N, C, Dv, M, GradStep{T0, __dmul_rn(2.0, lam), eta, T, M});
}
__global__ void __launch_bounds__(kFewWaves * 64)
scatter_few_step_kernel(const int32_t* __restrict__ perm, const int32_t* __restrict__ start, int64_t N, int C,
                        const double* __restrict__ Dv, int M, const float* __restrict__ T0, double lam, double eta,
                        double* __restrict__ T) {
  scatter_few_rows<double>(perm, start, N, C, Dv, M, GradStep{T0, __dmul_rn(2.0, lam), eta, T, M});
}

// -------------------------------------------------------------- assemble
// A = H + lambda I (lower triangle and diagonal; the strict upper triangle
// is never read), B = R + lambda T0 (in place in B).
__global__ void __launch_bounds__(256)
assemble_kernel(const int32_t* __restrict__ H, int64_t n, double lam, double* __restrict__ A,
                double* __restrict__ B, const float* __restrict__ T0, int64_t nb_total) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n * n; e += stride) {
    const int64_t i = e / n, j = e - (e / n) * n;
    if (j <= i) A[e] = (double)H[e] + (i == j ? lam : 0.0);
  }
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nb_total; e += stride)
    B[e] = __dadd_rn(B[e], __dmul_rn(lam, (double)T0[e]));
}

// ---------------------------------------------------------- factorisation
typedef double f64x4 __attribute__((ext_vector_type(4)));

// v's lane `from` (uniform), in every lane
__device__ __forceinline__ double lane_of(double v, int from) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, from);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), from);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Panel [j0, j0 + jb): the diagonal block's factor and the rows below it,
// L21 = A21 L11^-T, in one launch.  A wavefront holds the 32 rows of the
// diagonal block (lanes 0-31) and 32 rows below (lanes 32-63), a row of 32
// columns per lane, and factors the block along with its own rows: every
// wavefront repeats the block, none waits for another.  Right-looking, term
// k = column; after each column the row moves down one register, so that 8
// columns share one short loop body.  The block's factor goes to `diag`
// ([32][32], row-major): other wavefronts may still be reading the block, the
// trailing update's launch puts it in its place.  (No rows below: directly.)
// Bound: the chain of 32 square roots and divisions, about 250 cycles a column
// with the update of the next one: 14.5 us, against 21 us for the block in one
// workgroup with two barriers a column and then 18 us for the rows (21 us with
// the factors through readlane).
//
// The next pivot is lane j + 1's own value, so its square root starts at once;
// the column's other factors go round through LDS (s_c, aligned to the column,
// so they are read 16 bytes at a time, the same address in every lane).
// `root`: the square root of column j's pivot, kept from column to column.
template <int W>
__device__ __forceinline__ void panel_columns(double (&x)[kNB], double& root, int j, int j1, int lane, double* s_out,
                                              double* s_c) {
#pragma unroll 1
  for (; j < j1; ++j) {
    const double v = lane == j ? root : __ddiv_rn(x[0], root);
    s_out[lane * (kNB + 1) + j] = v;
    s_c[(lane - j - 1) & 63] = v;   // lane j + q at q - 1
    root = __dsqrt_rn(lane_of(__fma_rn(-v, v, x[1]), j + 1));
    // (the wavefront's own LDS, in order)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 1; q <= W; ++q) x[q - 1] = __fma_rn(-v, s_c[q - 1], x[q]);
    __builtin_amdgcn_wave_barrier();
  }
}

constexpr int kPanelWaves = 2;
__global__ void __launch_bounds__(kPanelWaves * 64)
panel_kernel(double* __restrict__ A, int64_t n, int j0, int jb, double* __restrict__ diag) {
  __shared__ double s_out[kPanelWaves][64 * (kNB + 1)];
  __shared__ __attribute__((aligned(16))) double s_col[kPanelWaves][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t w = (int64_t)blockIdx.x * kPanelWaves + wave;
  const int64_t below = (int64_t)j0 + jb + w * 32;   // first own row
  if (w > 0 && below >= n) return;
  const bool top = lane < 32;
  const int64_t row = top ? j0 + lane : below + lane - 32;
  const bool ok = top ? lane < jb : row < n;
  const double* ar = A + (ok ? row : j0) * n + j0;
  double x[kNB];
#pragma unroll
  for (int j = 0; j < kNB; ++j) x[j] = ok && j < jb && (!top || j <= lane) ? ar[j] : 0.0;
  double* so = s_out[wave];
  double* sc = s_col[wave];
  double root = __dsqrt_rn(lane_of(x[0], 0));
  panel_columns<31>(x, root, 0, 8, lane, so, sc);
  panel_columns<23>(x, root, 8, 16, lane, so, sc);
  if (jb > 16) {
    panel_columns<15>(x, root, 16, 24, lane, so, sc);
    panel_columns<7>(x, root, 24, 32, lane, so, sc);
  }
  // (a wavefront's own LDS, in order)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const bool only = (int64_t)j0 + jb >= n;
  for (int e = lane; e < 64 * kNB; e += 64) {
    const int r = e / kNB, j = e % kNB;
    const double v = so[r * (kNB + 1) + j];
    if (r < 32) {
      if (w == 0 && r < jb && j <= r) {
        if (only) A[(j0 + r) * n + j0 + j] = v;
        else diag[r * kNB + j] = v;
      }
    } else if (below + r - 32 < n && j < jb) {
      A[(below + r - 32) * n + j0 + j] = v;
    }
  }
}

// Trailing update: A[i][q] -= sum_{k in panel, ascending} L[i][k] L[q][k] for
// j0 + 32 <= q <= i < n (a panel with rows below it has all 32 columns); a 32 x
// 32 tile per workgroup (lower tiles only), 16 x 16 per wavefront, on the fp64
// matrix instruction: it takes its 4 terms k ascending, one fused multiply-add
// each (found equal to that chain bit for bit), so a tile's 32 terms are the
// unblocked algorithm's.  Lane l holds row (or column) l % 16 and term l / 16
// of the operands, column l % 16 and rows l / 16 + 4 r of the result; all loads
// go out together and no LDS is used: 4.6-7.6 us for n = 1024 against 7.5-10
// staged through LDS with 4 chains a thread.
__global__ void __launch_bounds__(256)
syrk_kernel(double* __restrict__ A, int64_t n, int j0, const double* __restrict__ diag) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // tile (ti, tq), ti >= tq, from the linear block index
  int ti = 0;
  const int b = blockIdx.x;
  while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
  const int tq = b - ti * (ti + 1) / 2;
  const int64_t s = (int64_t)j0 + kNB;
  if (b == 0)   // the diagonal block's factor into its place
    for (int e = threadIdx.x; e < kNB * kNB; e += 256) {
      const int i = e / kNB, j = e % kNB;
      if (j <= i) A[(j0 + i) * n + j0 + j] = diag[e];
    }
  const int64_t i0 = s + (int64_t)ti * kNB + 16 * (wave >> 1), q0 = s + (int64_t)tq * kNB + 16 * (wave & 1);
  if (i0 >= n || q0 > i0 + 15) return;   // (n is a multiple of 16)
  const int lr = lane & 15, lk = lane >> 4;
  const double* li = A + (i0 + lr) * n + j0 + lk;
  const double* lq = A + (q0 + lr) * n + j0 + lk;
  double va[kNB / 4], vb[kNB / 4];
  f64x4 c;
#pragma unroll
  for (int k = 0; k < kNB / 4; ++k) {
    va[k] = li[4 * k];
    vb[k] = lq[4 * k];
  }
  double* out = A + (i0 + lk) * n + q0 + lr;
#pragma unroll
  for (int r = 0; r < 4; ++r) c[r] = out[4 * r * n];
#pragma unroll
  for (int k = 0; k < kNB / 4; ++k) c = __builtin_amdgcn_mfma_f64_16x16x4f64(-va[k], vb[k], c, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (q0 + lr <= i0 + lk + 4 * r) out[4 * r * n] = c[r];
}

// ------------------------------------------------------------------ solves
// B [n][M] in place.  Forward: z_i = (b_i - sum_{k < i} L[i][k] z_k) / L[i][i],
// k ascending; backward: t_i = (z_i - sum_{k > i} L[k][i] t_k) / L[i][i], k
// descending.  Blocks of 32 rows; launch `i0` takes the terms of block i0
// (solved) to every row block still to come, 32 rows x 64 columns per
// workgroup, and the workgroups of the next block solve it at once, so a block
// costs one launch.  The terms go through the fp64 matrix instruction (k
// ascending inside it; the backward pass hands it the terms in reverse).
// i0 < 0: no terms, the first block is solved.
//
// Bound: launches and the solve's chain of 32 divisions: 11 us a block (n 1024,
// 512 columns) against 23 us for a launch of the solve and one of the terms.
constexpr int kTvCols = 64;

template <int W>
__device__ __forceinline__ void solve_rows(double (&x)[kNB], int i, int i1, const double (*s_l)[kNB], const double* s_d,
                                           double* __restrict__ out, int64_t step, bool ok) {
#pragma unroll 1
  for (; i < i1; ++i) {
    double l[W];   // (read before the division, which they do not wait for)
#pragma unroll
    for (int q = 0; q < W; ++q) l[q] = s_l[i][q];
    const double v = __ddiv_rn(x[0], s_d[i]);
    if (ok) out[i * step] = v;
#pragma unroll
    for (int q = 1; q <= W; ++q) x[q - 1] = __fma_rn(-l[q - 1], v, x[q]);
  }
}

template <bool FWD>
__global__ void __launch_bounds__(256)
trsv_kernel(const double* __restrict__ A, int64_t n, double* __restrict__ B, int M, int64_t i0, int ib, int64_t next0) {
  __shared__ double s_z[kNB][kTvCols];
  __shared__ __attribute__((aligned(16))) double s_l[kNB][kNB];   // [i][q - 1]: the factor of unknown i in unknown i + q
  __shared__ double s_d[kNB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntm = (M + kTvCols - 1) / kTvCols;
  // row blocks: forward next0, next0 + 32, ...; backward next0, next0 - 32, ...
  const int64_t r0 = FWD ? next0 + (int64_t)(blockIdx.x / ntm) * kNB : next0 - (int64_t)(blockIdx.x / ntm) * kNB;
  const int64_t m0 = (int64_t)(blockIdx.x % ntm) * kTvCols;
  const bool solve = r0 == next0;   // uniform
  const int rb = (int)(n - r0 < kNB ? n - r0 : kNB);   // 16 or 32 rows
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t col = m0 + 16 * wave + lr;
  const bool cok = col < M;
  const int64_t cc = cok ? col : M - 1;
  // every load first: the terms' operands, the rows, and for the solve the
  // block's factor (unknown i of the block is row i forward, row rb - 1 - i
  // backward)
  f64x4 c[2];
  double va[2][kNB / 4], vb[kNB / 4], f[kNB * kNB / 256], fd = 1.0;
  double* out = B + (r0 + lk) * M + cc;
#pragma unroll
  for (int k = 0; k < kNB / 4; ++k) {
    const int t = FWD ? 4 * k + lk : ib - 1 - (4 * k + lk);   // term: row i0 + t of the solved block
    const bool tok = i0 >= 0 && t >= 0 && t < ib;
    const int64_t gk = tok ? i0 + t : 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t gr = 16 * h < rb ? r0 + 16 * h + lr : r0;
      va[h][k] = tok ? (FWD ? A[gr * n + gk] : A[gk * n + gr]) : 0.0;
    }
    vb[k] = tok ? B[gk * (int64_t)M + cc] : 0.0;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) c[h][r] = 16 * h < rb ? out[(16 * h + 4 * r) * (int64_t)M] : 0.0;
  if (solve) {
#pragma unroll
    for (int u = 0; u < kNB * kNB / 256; ++u) {
      const int e = tid + 256 * u, i = e / kNB, q = e % kNB + 1;
      f[u] = i + q >= rb ? 0.0
             : FWD       ? A[(r0 + i + q) * n + r0 + i]
                         : A[(r0 + rb - 1 - i) * n + r0 + rb - 1 - i - q];
    }
    if (tid < rb) fd = A[(r0 + (FWD ? tid : rb - 1 - tid)) * (n + 1)];
  }
  if (i0 >= 0) {
#pragma unroll
    for (int k = 0; k < kNB / 4; ++k)
      if (4 * k < ib)
#pragma unroll
        for (int h = 0; h < 2; ++h) c[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(-va[h][k], vb[k], c[h], 0, 0, 0);
  }
  if (solve) {
#pragma unroll
    for (int u = 0; u < kNB * kNB / 256; ++u) s_l[(tid + 256 * u) / kNB][(tid + 256 * u) % kNB] = f[u];
    if (tid < kNB) s_d[tid] = fd;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (solve)
        s_z[16 * h + lk + 4 * r][16 * wave + lr] = c[h][r];
      else if (cok && 16 * h < rb)
        out[(16 * h + 4 * r) * (int64_t)M] = c[h][r];
    }
  if (!solve) return;
  __syncthreads();
  if (wave != 0) return;
  double x[kNB];
#pragma unroll
  for (int i = 0; i < kNB; ++i) x[i] = i < rb ? s_z[FWD ? i : rb - 1 - i][lane] : 0.0;
  const int64_t m = m0 + lane;
  const bool ok = m < M;
  double* z = B + (FWD ? r0 : r0 + rb - 1) * (int64_t)M + (ok ? m : 0);
  const int64_t step = FWD ? M : -(int64_t)M;
  solve_rows<31>(x, 0, 8, s_l, s_d, z, step, ok);
  solve_rows<23>(x, 8, 16, s_l, s_d, z, step, ok);
  if (rb > 16) {
    solve_rows<15>(x, 16, 24, s_l, s_d, z, step, ok);
    solve_rows<7>(x, 24, 32, s_l, s_d, z, step, ok);
  }
}

// ------------------------------------------- nonlinear output: gradient descent
// z_n = (sum_c T[c][idx[n][c]][.], c ascending) + b.  One wavefront per row,
// lanes over columns; the row's indices are uniform (scalar loads).
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v = __dadd_rn(v, __shfl_xor(v, o));
  return v;
}

// Softmax of the row held in out[0..M) (in place): maximum subtracted, exp,
// sum, division.
__device__ void softmax_row_inplace(double* __restrict__ out, int M, int lane) {
  double mx = -__builtin_inf();
  for (int m = lane; m < M; m += 64) mx = fmax(mx, out[m]);
  mx = wave_max(mx);
  double sum = 0.0;
  for (int m = lane; m < M; m += 64) {
    const double e = exp(__dsub_rn(out[m], mx));
    out[m] = e;
    sum = __dadd_rn(sum, e);
  }
  sum = wave_sum(sum);
  for (int m = lane; m < M; m += 64) out[m] = __ddiv_rn(out[m], sum);
}

// P = sigma(Y + b): ReLU (act 2) or row softmax (acts 3 and 4), in double
__global__ void __launch_bounds__(256)
target_kernel(const float* __restrict__ Y, int64_t N, int M, const float* __restrict__ bias, int act,
              double* __restrict__ P) {
  const int lane = threadIdx.x & 63;
  for (int64_t n = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); n < N; n += (int64_t)gridDim.x * 4) {
    double* pr = P + n * M;
    for (int m = lane; m < M; m += 64) {
      const double z = __dadd_rn((double)Y[n * M + m], bias ? (double)bias[m] : 0.0);
      pr[m] = (act == 2) ? (z > 0.0 ? z : 0.0) : z;
    }
    if (act >= 3) softmax_row_inplace(pr, M, lane);
  }
}

// The sums over the codebooks, c ascending, of row n's table rows at columns
// lane, lane + 64, ... (J of them; columns past M read column M - 1): the
// indices come 64 codebooks at a time, one per lane, and are handed out
// through readlane, so a table row's address is uniform and 8 codebooks' loads
// are in flight.  n and m0 are uniform and all 64 lanes are active: readlane
// reads a lane's register also where the lane is not, and then finds what an
// earlier call left there.
template <int J>
__device__ __forceinline__ void gather_row(const uint8_t* __restrict__ ir, int C, const double* __restrict__ T, int M,
                                           int m0, int lane, double (&s)[J]) {
  int col[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    s[j] = 0.0;
    col[j] = min(m0 + lane + 64 * j, M - 1);
  }
  for (int c0 = 0; c0 < C; c0 += 64) {
    const int key = c0 + lane < C ? (int)(ir[c0 + lane] & 15) : 0;
    const double* tc = T + (int64_t)c0 * kK * M;
    const int nc = min(64, C - c0);
    constexpr int kU = 8;
    for (int c = 0; c < nc; c += kU) {
      double v[kU][J];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int cu = min(c + u, nc - 1);
        const double* row = tc + (int64_t)(cu * kK + __builtin_amdgcn_readlane(key, cu)) * M;
#pragma unroll
        for (int j = 0; j < J; ++j) v[u][j] = row[col[j]];
      }
#pragma unroll
      for (int u = 0; u < kU; ++u)
        if (c + u < nc) {
#pragma unroll
          for (int j = 0; j < J; ++j) s[j] = __dadd_rn(s[j], v[u][j]);
        }
    }
  }
}

// D = dObjective / dz per row: ReLU 2 (relu(z) - P) [z > 0]; softmax with the
// KL divergence softmax(z) - P; softmax with the squared error 2 p (d - s),
// p = softmax(z), d = p - P, s = sum_m d_m p_m (the softmax Jacobian
// diag(p) - p p^T applied to 2 d).  One wavefront per row; rows of at most
// 64 J columns stay in registers, each lane's columns in the same order as
// through memory.  Bound: the table rows out of the L2, 8 bytes per (row,
// codebook, column) (16,384 x 32 x 64: 44 -> 26 us, 10 TB/s).
template <int J>
__global__ void __launch_bounds__(256)
resid_reg_kernel(const uint8_t* __restrict__ idx, int64_t N, int C, const double* __restrict__ T, int M,
                 const float* __restrict__ bias, int act, const double* __restrict__ P, double* __restrict__ D) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int64_t n = (int64_t)blockIdx.x * 4 + wave; n < N; n += (int64_t)gridDim.x * 4) {
    double z[J], p[J];
#pragma unroll
    for (int j = 0; j < J; ++j) p[j] = P[n * M + min(lane + 64 * j, M - 1)];
    gather_row<J>(idx + n * C, C, T, M, 0, lane, z);
#pragma unroll
    for (int j = 0; j < J; ++j) z[j] = __dadd_rn(z[j], bias ? (double)bias[min(lane + 64 * j, M - 1)] : 0.0);
    if (act == 2) {
#pragma unroll
      for (int j = 0; j < J; ++j) z[j] = z[j] > 0.0 ? __dmul_rn(2.0, __dsub_rn(z[j], p[j])) : 0.0;
    } else {
      double mx = -__builtin_inf(), sum = 0.0;
#pragma unroll
      for (int j = 0; j < J; ++j)
        if (lane + 64 * j < M) mx = fmax(mx, z[j]);
      mx = wave_max(mx);
#pragma unroll
      for (int j = 0; j < J; ++j)
        if (lane + 64 * j < M) {
          z[j] = exp(__dsub_rn(z[j], mx));
          sum = __dadd_rn(sum, z[j]);
        }
      sum = wave_sum(sum);
#pragma unroll
      for (int j = 0; j < J; ++j) z[j] = __ddiv_rn(z[j], sum);
      if (act == 3) {
#pragma unroll
        for (int j = 0; j < J; ++j) z[j] = __dsub_rn(z[j], p[j]);
      } else {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j)
          if (lane + 64 * j < M) s = __dadd_rn(s, __dmul_rn(__dsub_rn(z[j], p[j]), z[j]));
        s = wave_sum(s);
#pragma unroll
        for (int j = 0; j < J; ++j) z[j] = __dmul_rn(2.0, __dmul_rn(z[j], __dsub_rn(__dsub_rn(z[j], p[j]), s)));
      }
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (lane + 64 * j < M) D[n * M + lane + 64 * j] = z[j];
  }
}

// the same for rows of any width: the row goes through D
__global__ void __launch_bounds__(256)
resid_kernel(const uint8_t* __restrict__ idx, int64_t N, int C, const double* __restrict__ T, int M,
             const float* __restrict__ bias, int act, const double* __restrict__ P, double* __restrict__ D) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int64_t n = (int64_t)blockIdx.x * 4 + wave; n < N; n += (int64_t)gridDim.x * 4) {
    double* dr = D + n * M;
    const double* pr = P + n * M;
    for (int m0 = 0; m0 < M; m0 += 64) {   // uniform: every lane takes part in gather_row
      const int m = m0 + lane;
      double s[1];
      gather_row<1>(idx + n * C, C, T, M, m0, lane, s);
      if (m < M) {
        const double z = __dadd_rn(s[0], bias ? (double)bias[m] : 0.0);
        dr[m] = (act == 2) ? (z > 0.0 ? __dmul_rn(2.0, __dsub_rn(z, pr[m])) : 0.0) : z;
      }
    }
    if (act == 3) {
      softmax_row_inplace(dr, M, lane);
      for (int m = lane; m < M; m += 64) dr[m] = __dsub_rn(dr[m], pr[m]);
    } else if (act == 4) {
      softmax_row_inplace(dr, M, lane);
      double s = 0.0;
      for (int m = lane; m < M; m += 64) s = __dadd_rn(s, __dmul_rn(__dsub_rn(dr[m], pr[m]), dr[m]));
      s = wave_sum(s);
      for (int m = lane; m < M; m += 64) {
        const double p = dr[m];
        dr[m] = __dmul_rn(2.0, __dmul_rn(p, __dsub_rn(__dsub_rn(p, pr[m]), s)));
      }
    }
  }
}

__global__ void __launch_bounds__(256) copy_f32_f64_kernel(const float* __restrict__ a, double* __restrict__ b,
                                                           int64_t total) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256)
    b[e] = (double)a[e];
}

unsigned grid_1d(int64_t total, int per) {
  int64_t g = (total + per - 1) / per;
  if (g < 1) g = 1;
  if (g > 65536) g = 65536;
  return (unsigned)g;
}

}  // namespace

hipError_t launch_gram(const uint8_t* idx, int64_t N, int C, int32_t* H, int cus, hipStream_t stream) {
  const int64_t n16 = (int64_t)C * kK;
  hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_1d(n16 * n16, 256)), dim3(256), 0, stream, H, n16 * n16);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || N == 0) return e;
  const int nbc = (C + kGB - 1) / kGB;
  const int64_t npair = (int64_t)nbc * nbc;
  // about four workgroups per CU in all, chunks of at least 256 rows
  int64_t chunks = ((int64_t)4 * cus + npair - 1) / npair;
  const int64_t max_chunks = (N + 255) / 256;
  if (chunks > max_chunks) chunks = max_chunks;
  if (chunks < 1) chunks = 1;
  const int64_t chunk_rows = (N + chunks - 1) / chunks;
  chunks = (N + chunk_rows - 1) / chunk_rows;
  hipLaunchKernelGGL(gram_kernel, dim3((unsigned)(npair * chunks)), dim3(256), 0, stream, idx, N, C, nbc,
                     chunk_rows, H);
  return hipGetLastError();
}

hipError_t launch_partition(const uint8_t* idx, int64_t N, int C, int32_t* perm, int32_t* start,
                            hipStream_t stream) {
  hipLaunchKernelGGL(partition_kernel, dim3((unsigned)C), dim3(kPartWaves * 64), 0, stream, idx, N, C, perm, start);
  return hipGetLastError();
}

hipError_t launch_scatter(const uint8_t* idx, int64_t N, int C, const float* Y, int M, double* R,
                          int32_t* perm, int32_t* start, hipStream_t stream) {
  hipError_t e = launch_partition(idx, N, C, perm, start, stream);
  if (e != hipSuccess) return e;
  if (few_rows_sum(N, C, M))
    hipLaunchKernelGGL(scatter_few_kernel, dim3(few_rows_grid(C, M)), dim3(kFewWaves * 64), 0, stream, perm, start, N,
                       C, Y, M, R);
  else
    hipLaunchKernelGGL(scatter_kernel, dim3(scatter_grid(C, M, kScCols)), dim3(kScWaves * 64), 0, stream, perm, start,
                       N, C, Y, M, R);
  return hipGetLastError();
}

hipError_t launch_fit_ridge(const uint8_t* idx, int64_t N, int C, const float* Y, int M, const float* T0,
                            double lam, double* T, int32_t* H, double* A, int32_t* perm, int32_t* start,
                            int cus, hipStream_t stream) {
  const int64_t n = (int64_t)C * kK;
  hipError_t e = launch_gram(idx, N, C, H, cus, stream);
  if (e != hipSuccess) return e;
  e = launch_scatter(idx, N, C, Y, M, T, perm, start, stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(assemble_kernel, dim3(grid_1d(n * n, 256)), dim3(256), 0, stream, H, n, lam, A, T, T0,
                     n * M);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // (the counts are not read any more: their array holds a panel's diagonal
  // block, 8 KB, when the panel has rows below it, n >= 48)
  double* diag = reinterpret_cast<double*>(H);
  for (int j0 = 0; j0 < n; j0 += kNB) {
    const int jb = (int)((n - j0) < kNB ? (n - j0) : kNB);
    const int64_t below = n - j0 - jb;
    const int64_t waves = below > 0 ? (below + 31) / 32 : 1;
    hipLaunchKernelGGL(panel_kernel, dim3((unsigned)((waves + kPanelWaves - 1) / kPanelWaves)), dim3(kPanelWaves * 64), 0,
                       stream, A, n, j0, jb, diag);
    if (below > 0) {
      const int64_t tiles = (below + kNB - 1) / kNB;
      hipLaunchKernelGGL(syrk_kernel, dim3((unsigned)(tiles * (tiles + 1) / 2)), dim3(256), 0, stream, A, n, j0, diag);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int64_t ntm = (M + kTvCols - 1) / kTvCols;
  const int64_t last = ((n - 1) / kNB) * kNB;
  for (int64_t i0 = -kNB; i0 < last; i0 += kNB) {   // forward: block i0's terms, block i0 + 32 solved
    const int64_t next0 = i0 + kNB;
    const int64_t blocks = i0 < 0 ? 1 : (n - next0 + kNB - 1) / kNB;
    hipLaunchKernelGGL(trsv_kernel<true>, dim3((unsigned)(blocks * ntm)), dim3(256), 0, stream, A, n, T, M, i0, kNB,
                       next0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  for (int64_t next0 = last; next0 >= 0; next0 -= kNB) {   // backward: block next0 + 32's terms, block next0 solved
    const int64_t i0 = next0 == last ? -1 : next0 + kNB;
    const int ib = (int)(i0 >= 0 && n - i0 < kNB ? n - i0 : kNB);
    const int64_t blocks = i0 < 0 ? 1 : next0 / kNB + 1;
    hipLaunchKernelGGL(trsv_kernel<false>, dim3((unsigned)(blocks * ntm)), dim3(256), 0, stream, A, n, T, M, i0, ib,
                       next0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_fit_gd(const uint8_t* idx, int64_t N, int C, const float* Y, int M, const float* bias, int act,
                         const float* T0, double lam, double eta, int iters, double* T, double* P, double* D,
                         int32_t* perm, int32_t* start, hipStream_t stream) {
  const int64_t total = (int64_t)C * kK * M;
  hipLaunchKernelGGL(copy_f32_f64_kernel, dim3(grid_1d(total, 256)), dim3(256), 0, stream, T0, T, total);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || iters == 0) return e;
  if ((e = launch_partition(idx, N, C, perm, start, stream)) != hipSuccess) return e;
  const unsigned rows = grid_1d((N + 3) / 4, 1);   // 4 rows per workgroup, rows looped past 65536 groups
  if (N > 0) {
    hipLaunchKernelGGL(target_kernel, dim3(rows), dim3(256), 0, stream, Y, N, M, bias, act, P);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  for (int it = 0; it < iters; ++it) {
    if (N > 0) {
      auto resid = M <= 64 ? resid_reg_kernel<1> : M <= 128 ? resid_reg_kernel<2> : M <= 256 ? resid_reg_kernel<4>
                                                                                             : resid_kernel;
      hipLaunchKernelGGL(resid, dim3(rows), dim3(256), 0, stream, idx, N, C, T, M, bias, act, P, D);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const bool few = few_rows_step(N, C, M);
    auto step = few ? scatter_few_step_kernel : step_cols(M) == 16 ? scatter_step_kernel<16> : scatter_step_kernel<64>;
    const unsigned blocks = few ? few_rows_grid(C, M) : scatter_grid(C, M, step_cols(M));
    hipLaunchKernelGGL(step, dim3(blocks), dim3((few ? kFewWaves : kScWaves) * 64), 0, stream, perm, start, N, C, D, M,
                       T0, lam, eta, T);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mdn
