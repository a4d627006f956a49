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
//           blocked right-looking Cholesky factorisation (panels of 32:
//           diagonal block in one workgroup, the rows below it, then the
//           trailing update), then blocked forward and backward substitution
//           over the M columns of B, in place.
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
// rows of bucket k, start[c][k] the bucket starts (start[c][16] = N).  Each
// codebook's list is followed by 128 entries of row 0, read (and ignored) past the last
// bucket.
constexpr int kPermPad = 128;

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
  int32_t* pc = perm + (int64_t)c * (N + kPermPad);
  if (threadIdx.x < kPermPad) pc[N + threadIdx.x] = 0;
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
// The sum of a bucket is one chain of dependent adds (4.5 cycles each), and
// buckets are uneven (the largest of a random tree's 16 holds about half of
// the rows), so the adding wavefront does nothing else.  Bound: on small
// layers that chain, on large ones the L2, which reads every row once per
// codebook.  Column tiles go to XCDs (workgroup b runs on XCD b % 8): with a
// number of tiles that divides 8, or a multiple of 8, each XCD reads its own
// columns only, and TC is such that they fit its 4 MB L2 at the training sets'
// sizes; else the tiles are taken one after the other.
// Measured against one wavefront per codebook with its 16 buckets in turn:
// 16,384 rows, 32 codebooks x 64 columns of doubles 554 -> 79 us (largest
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
    const int32_t* pc = perm + (int64_t)c * (N + kPermPad);
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

constexpr int kScCols = 64;                                            // columns of floats per workgroup
constexpr int step_cols(int M) { return M <= 128 ? 16 : 32; }          // of doubles: 8 tiles, or the fewer LDS accesses
unsigned scatter_grid(int C, int M, int cols) { return (unsigned)(C * kK * ((M + cols - 1) / cols)); }

__global__ void __launch_bounds__(kScWaves * 64)
scatter_kernel(const int32_t* __restrict__ perm, const int32_t* __restrict__ start, int64_t N, int C,
               const float* __restrict__ Y, int M, double* __restrict__ R) {
  scatter_bucket<float, kScCols>(perm, start, N, C, Y, M, [&](int64_t r, int m, double v) { R[r * M + m] = v; });
}

// The gradient step on the sums just made: T = T - eta (R + 2 lambda (T - T0))
template <int TC>
__global__ void __launch_bounds__(kScWaves * 64)
scatter_step_kernel(const int32_t* __restrict__ perm, const int32_t* __restrict__ start, int64_t N, int C,
                    const double* __restrict__ Dv, int M, const float* __restrict__ T0, double lam, double eta,
                    double* __restrict__ T) {
  const double two_lam = __dmul_rn(2.0, lam);
  scatter_bucket<double, TC>(perm, start, N, C, Dv, M, [&](int64_t r, int m, double v) {
    const int64_t e = r * M + m;
    const double g = __dadd_rn(v, __dmul_rn(two_lam, __dsub_rn(T[e], (double)T0[e])));
    T[e] = __dsub_rn(T[e], __dmul_rn(eta, g));
  });
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
// diagonal block [j0, j0 + jb) of the panel: unblocked right-looking in LDS
__global__ void __launch_bounds__(256) potrf_diag_kernel(double* __restrict__ A, int64_t n, int j0, int jb) {
  __shared__ double a[kNB][kNB + 1];
  const int tid = threadIdx.x;
  for (int e = tid; e < kNB * kNB; e += 256) {
    const int i = e / kNB, j = e % kNB;
    a[i][j] = (i < jb && j <= i) ? A[(j0 + i) * n + j0 + j] : 0.0;
  }
  __syncthreads();
  for (int j = 0; j < jb; ++j) {
    if (tid == 0) a[j][j] = __dsqrt_rn(a[j][j]);
    __syncthreads();
    const double d = a[j][j];
    for (int i = j + 1 + tid; i < jb; i += 256) a[i][j] = __ddiv_rn(a[i][j], d);
    __syncthreads();
    // update of the columns right of j: entry (i, q), j < q <= i, term k = j
    for (int e = tid; e < kNB * kNB; e += 256) {
      const int i = e / kNB, q = e % kNB;
      if (q > j && q <= i && i < jb) a[i][q] = __fma_rn(-a[i][j], a[q][j], a[i][q]);
    }
    __syncthreads();
  }
  for (int e = tid; e < kNB * kNB; e += 256) {
    const int i = e / kNB, j = e % kNB;
    if (i < jb && j <= i) A[(j0 + i) * n + j0 + j] = a[i][j];
  }
}

// rows [j0 + jb, n) of the panel: L21 = A21 L11^-T, one row per thread
__global__ void __launch_bounds__(256) trsm_panel_kernel(double* __restrict__ A, int64_t n, int j0, int jb) {
  __shared__ double l[kNB][kNB + 1];
  const int tid = threadIdx.x;
  for (int e = tid; e < kNB * kNB; e += 256) {
    const int i = e / kNB, j = e % kNB;
    l[i][j] = (i < jb && j <= i) ? A[(j0 + i) * n + j0 + j] : 0.0;
  }
  __syncthreads();
  const int64_t row = (int64_t)j0 + jb + (int64_t)blockIdx.x * 256 + tid;
  if (row >= n) return;
  double* ar = A + row * n + j0;
  double x[kNB];
#pragma unroll
  for (int j = 0; j < kNB; ++j) x[j] = j < jb ? ar[j] : 0.0;
#pragma unroll
  for (int j = 0; j < kNB; ++j) {
    if (j < jb) {
      x[j] = __ddiv_rn(x[j], l[j][j]);
#pragma unroll
      for (int q = j + 1; q < kNB; ++q) x[q] = __fma_rn(-x[j], l[q][j], x[q]);
    }
  }
#pragma unroll
  for (int j = 0; j < kNB; ++j)
    if (j < jb) ar[j] = x[j];
}

// trailing update: A[i][q] -= sum_{k in panel, ascending} L[i][k] L[q][k] for
// j0 + jb <= q <= i < n; a 32 x 32 tile per workgroup (lower tiles only)
__global__ void __launch_bounds__(256) syrk_kernel(double* __restrict__ A, int64_t n, int j0, int jb) {
  __shared__ double li[kNB][kNB + 1];
  __shared__ double lq[kNB][kNB + 1];
  const int tid = threadIdx.x;
  // tile (ti, tq), ti >= tq, from the linear block index
  int ti = 0;
  const int b = blockIdx.x;
  while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
  const int tq = b - ti * (ti + 1) / 2;
  const int64_t s = (int64_t)j0 + jb;
  const int64_t i0 = s + (int64_t)ti * kNB, q0 = s + (int64_t)tq * kNB;
  for (int e = tid; e < kNB * kNB; e += 256) {
    const int r = e / kNB, k = e % kNB;
    li[r][k] = (i0 + r < n && k < jb) ? A[(i0 + r) * n + j0 + k] : 0.0;
    lq[r][k] = (q0 + r < n && k < jb) ? A[(q0 + r) * n + j0 + k] : 0.0;
  }
  __syncthreads();
  const int ty = tid / 16, tx = tid % 16;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int r = ty + 16 * a, q = tx + 16 * c;
      const int64_t gi = i0 + r, gq = q0 + q;
      if (gi < n && gq <= gi) {
        double v = A[gi * n + gq];
        for (int k = 0; k < jb; ++k) v = __fma_rn(-li[r][k], lq[q][k], v);
        A[gi * n + gq] = v;
      }
    }
}

// ------------------------------------------------------------------ solves
// B [n][M] in place.  Forward: z_i = (b_i - sum_{k < i} L[i][k] z_k) / L[i][i],
// k ascending; backward: t_i = (z_i - sum_{k > i} L[k][i] t_k) / L[i][i], k
// descending.  Blocks of 32 rows; the diagonal block one column per thread,
// the update of the other rows as 32 x 64 tiles.
template <bool FWD>
__global__ void __launch_bounds__(256) trsv_diag_kernel(const double* __restrict__ A, int64_t n, double* __restrict__ B,
                                                         int M, int i0, int ib) {
  __shared__ double l[kNB][kNB + 1];
  const int tid = threadIdx.x;
  for (int e = tid; e < kNB * kNB; e += 256) {
    const int i = e / kNB, j = e % kNB;
    l[i][j] = (i < ib && j <= i) ? A[(i0 + i) * n + i0 + j] : 0.0;
  }
  __syncthreads();
  const int64_t m = (int64_t)blockIdx.x * 256 + tid;
  if (m >= M) return;
  double x[kNB];
#pragma unroll
  for (int i = 0; i < kNB; ++i) x[i] = i < ib ? B[(i0 + i) * (int64_t)M + m] : 0.0;
  if (FWD) {
#pragma unroll
    for (int i = 0; i < kNB; ++i) {
      if (i < ib) {
        x[i] = __ddiv_rn(x[i], l[i][i]);
#pragma unroll
        for (int q = i + 1; q < kNB; ++q) x[q] = __fma_rn(-l[q][i], x[i], x[q]);
      }
    }
  } else {
#pragma unroll
    for (int i = kNB - 1; i >= 0; --i) {
      if (i < ib) {
        x[i] = __ddiv_rn(x[i], l[i][i]);
#pragma unroll
        for (int q = 0; q < i; ++q) x[q] = __fma_rn(-l[i][q], x[i], x[q]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kNB; ++i)
    if (i < ib) B[(i0 + i) * (int64_t)M + m] = x[i];
}

// FWD: rows r >= i0 + ib get the block's terms, k ascending: b_r -= L[r][k] z_k.
// !FWD: rows r < i0 get them, k descending: b_r -= L[k][r] t_k.
template <bool FWD>
__global__ void __launch_bounds__(256) trsv_update_kernel(const double* __restrict__ A, int64_t n, double* __restrict__ B,
                                                           int M, int i0, int ib) {
  __shared__ double lr[kNB][kNB + 1];   // lr[r][k]: the coefficient of block row k in row r
  __shared__ double z[kNB][64];
  const int tid = threadIdx.x;
  const int ntm = (M + 63) / 64;
  const int64_t r0 = FWD ? (int64_t)i0 + ib + (int64_t)(blockIdx.x / ntm) * kNB : (int64_t)(blockIdx.x / ntm) * kNB;
  const int64_t rend = FWD ? n : i0;
  const int64_t m0 = (int64_t)(blockIdx.x % ntm) * 64;
  for (int e = tid; e < kNB * kNB; e += 256) {
    const int r = e / kNB, k = e % kNB;
    const int64_t gr = r0 + r;
    double v = 0.0;
    if (gr < rend && k < ib) v = FWD ? A[gr * n + i0 + k] : A[(i0 + k) * n + gr];
    lr[r][k] = v;
  }
  for (int e = tid; e < kNB * 64; e += 256) {
    const int k = e / 64, c = e % 64;
    z[k][c] = (k < ib && m0 + c < M) ? B[(i0 + k) * (int64_t)M + m0 + c] : 0.0;
  }
  __syncthreads();
  const int c = tid % 64;
  const int rr = tid / 64;   // rows rr, rr + 4, ..., 8 per thread
  if (m0 + c >= M) return;
#pragma unroll
  for (int a = 0; a < kNB / 4; ++a) {
    const int r = rr + 4 * a;
    const int64_t gr = r0 + r;
    if (gr >= rend) continue;
    double v = B[gr * (int64_t)M + m0 + c];
    if (FWD) {
      for (int k = 0; k < ib; ++k) v = __fma_rn(-lr[r][k], z[k][c], v);
    } else {
      for (int k = ib - 1; k >= 0; --k) v = __fma_rn(-lr[r][k], z[k][c], v);
    }
    B[gr * (int64_t)M + m0 + c] = v;
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
// are in flight.  n is uniform.
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
    for (int m = lane; m < M; m += 64) {
      double s[1];
      gather_row<1>(idx + n * C, C, T, M, m - lane, lane, s);
      const double z = __dadd_rn(s[0], bias ? (double)bias[m] : 0.0);
      dr[m] = (act == 2) ? (z > 0.0 ? __dmul_rn(2.0, __dsub_rn(z, pr[m])) : 0.0) : z;
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
  hipLaunchKernelGGL(scatter_kernel, dim3(scatter_grid(C, M, kScCols)), dim3(kScWaves * 64), 0, stream, perm, start, N,
                     C, Y, M, R);
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
  for (int j0 = 0; j0 < n; j0 += kNB) {
    const int jb = (int)((n - j0) < kNB ? (n - j0) : kNB);
    hipLaunchKernelGGL(potrf_diag_kernel, dim3(1), dim3(256), 0, stream, A, n, j0, jb);
    const int64_t below = n - j0 - jb;
    if (below > 0) {
      hipLaunchKernelGGL(trsm_panel_kernel, dim3(grid_1d(below, 256)), dim3(256), 0, stream, A, n, j0, jb);
      const int64_t tiles = (below + kNB - 1) / kNB;
      hipLaunchKernelGGL(syrk_kernel, dim3((unsigned)(tiles * (tiles + 1) / 2)), dim3(256), 0, stream, A, n, j0,
                         jb);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int ntm = (M + 63) / 64;
  for (int i0 = 0; i0 < n; i0 += kNB) {   // forward
    const int ib = (int)((n - i0) < kNB ? (n - i0) : kNB);
    hipLaunchKernelGGL(trsv_diag_kernel<true>, dim3(grid_1d(M, 256)), dim3(256), 0, stream, A, n, T, M, i0, ib);
    const int64_t below = n - i0 - ib;
    if (below > 0)
      hipLaunchKernelGGL(trsv_update_kernel<true>, dim3((unsigned)(((below + kNB - 1) / kNB) * ntm)), dim3(256), 0,
                         stream, A, n, T, M, i0, ib);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int64_t last = ((n - 1) / kNB) * kNB;
  for (int64_t i0 = last; i0 >= 0; i0 -= kNB) {   // backward
    const int ib = (int)((n - i0) < kNB ? (n - i0) : kNB);
    hipLaunchKernelGGL(trsv_diag_kernel<false>, dim3(grid_1d(M, 256)), dim3(256), 0, stream, A, n, T, M, (int)i0,
                       ib);
    if (i0 > 0)
      hipLaunchKernelGGL(trsv_update_kernel<false>, dim3((unsigned)(((i0 + kNB - 1) / kNB) * ntm)), dim3(256), 0,
                         stream, A, n, T, M, (int)i0, ib);
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
    auto step = step_cols(M) == 16 ? scatter_step_kernel<16> : scatter_step_kernel<32>;
    hipLaunchKernelGGL(step, dim3(scatter_grid(C, M, step_cols(M))), dim3(kScWaves * 64), 0, stream, perm,
                       start, N, C, D, M, T0, lam, eta, T);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mdn
