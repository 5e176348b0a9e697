// k_decor.hip -- correlation-reducing permutation of an LHS design (Sec. IV-B,
// LHS Step 2: the rows may be permuted by any rule; the paper points to
// Cholesky-based correlation control).  The M rows of the design are taken as
// M variables observed in N samples.  Their sample covariance C is factored
// C = L L^T, the scores Z = L^{-1} (X - mean) have identity sample covariance,
// and each row of X is rearranged so that its values take the ranks of the
// same row of Z (one pass of rank-based correlation control towards the
// identity).  A row keeps its values; only their assignment to samples
// changes, so an LHS row still holds one value per stratum.
//
// Steps on the stream, all FP64:
//   k_dc_mean    row means                        M workgroups
//   k_dc_cov     lower-triangle 64x64 tiles of C  x sample slices, then k_dc_cov_sum
//   k_dc_chol    Cholesky by 16-column blocks     one workgroup (M <= 1024)
//   k_dc_whiten  substitution by 16-row blocks    a wave per 16 samples
//   k_dc_rank_row             ranks in each row   buckets + prefix sums, O(N) expected;
//                workgroups per row in LDS, k_dc_range .. k_dc_rank for longer rows
//   k_dc_apply   rearrangement                    one thread per entry
// The products (covariance, trailing updates, substitution) run on the FP64 matrix
// cores, v_mfma_f64_16x16x4: lane l holds row l%16, column l/16 of A, row l/16,
// column l%16 of B, and rows 4 r + l/16 of column l%16 of the result (r = 0..3),
// so a result's register r is the B operand of step r of a product with it.
// 300 rows of 1e4 samples: 1.72 -> 0.58 ms for the whole design.
// Ranks order equal values by the lower sample index and always form a
// permutation, so every gather stays in bounds whatever the values are.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "decor_plan.hpp"
#include "fmc_internal.hpp"
#include "fmc_runtime.hpp"

namespace fmc {

namespace {

constexpr int kDcCovTile = 64;  // covariance tile edge (32x32 entries per wave)
constexpr int kDcChunk = 32;    // samples per LDS stage of the covariance
constexpr int kDcStride = 36;   // LDS row stride of the 32 samples (no bank conflicts)
constexpr int kDcCholThreads = 512;
// Longest rows ranked in LDS: two 32-bit words per entry, and with its value.
constexpr int64_t kDcRowMax = 20000, kDcRowValues = 10200;
constexpr int kDcRankThreads = 1024;
// Comparisons inside buckets, per entry of the row and workgroup, from which a row is
// sorted instead; workgroups of a row at most (k_dc_rank_row).
constexpr int kDcCrowd = 192, kDcRankSplit = 16;

// Static LDS of k_dc_rank_row; it and the arrays of the longest rows fit a CU's 160 KB.
constexpr size_t kDcRankStatic = kDcRankThreads / 64 * (2 * sizeof(double) + 2 * sizeof(int32_t));
static_assert(kDcRankStatic + kDcRowValues * sizeof(double) + (2 * kDcRowValues + 1) * sizeof(int32_t) <= 160 * 1024 &&
                  kDcRankStatic + (2 * kDcRowMax + 1) * sizeof(int32_t) <= 160 * 1024,
              "LDS of the rows ranked in LDS");

typedef double d4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4v mma(double a, double b, d4v c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// value of v in lane i of each row of 16 lanes (i a constant after unrolling)
__device__ __forceinline__ double row_lane(double v, int i) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  switch (i) {
#define FMC_X(K) \
  case K:        \
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, 0x150 + K, 0xF, 0xF, false), \
                            __builtin_amdgcn_update_dpp(0, lo, 0x150 + K, 0xF, 0xF, false));
    FMC_X(0) FMC_X(1) FMC_X(2) FMC_X(3) FMC_X(4) FMC_X(5) FMC_X(6) FMC_X(7)
    FMC_X(8) FMC_X(9) FMC_X(10) FMC_X(11) FMC_X(12) FMC_X(13) FMC_X(14) FMC_X(15)
#undef FMC_X
  }
  return v;
}

__global__ void __launch_bounds__(256) k_dc_mean(int64_t N, const double* __restrict__ X,
                                                 double* __restrict__ mean) {
  const double* x = X + (int64_t)blockIdx.x * N;
  double s = 0.0;
  for (int64_t n = threadIdx.x; n < N; n += 256) s += x[n];
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) mean[blockIdx.x] = red[0] / (double)N;
}

// Partial sample cross-products of the centred rows over one slice of the
// samples (blockIdx.y), for one 64x64 tile (ta, tb), ta >= tb, of C
// (blockIdx.x enumerates the lower-triangle tiles).  Wave w holds the 32x32 entries
// (w / 2, w % 2) as four matrix tiles; chunks of 32 samples are staged in LDS.
// (As 4x4 entries per thread on the vector units the products took 90 us at 300
// rows of 1e4 samples; 48 us here.)
__global__ void __launch_bounds__(256) k_dc_cov(int M, int64_t N, int64_t per,
                                                const double* __restrict__ X,
                                                const double* __restrict__ mean,
                                                double* __restrict__ P) {
  int t = blockIdx.x, ta = 0;
  while (t > ta) {
    t -= ta + 1;
    ++ta;
  }
  const int tb = t;
  const int64_t nb0 = (int64_t)blockIdx.y * per;
  const int64_t nb1 = std::min<int64_t>(N, nb0 + per);
  const int wave = threadIdx.x / 64, l = threadIdx.x % 64, c = l & 15, g = l >> 4;
  const int wa = 32 * (wave / 2), wb = 32 * (wave % 2);
  __shared__ double sa[kDcCovTile][kDcStride], sb[kDcCovTile][kDcStride];
  d4v acc[2][2] = {};
  // a thread's entries of a chunk: sample tid % 32 of rows tid / 32 + 8 u, loaded a
  // chunk ahead
  constexpr int kU = kDcCovTile * kDcChunk / 256;
  const int kk = threadIdx.x % kDcChunk, r0 = threadIdx.x / kDcChunk;
  double xa[kU], xb[kU], ma[kU], mb[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int ra = ta * kDcCovTile + r0 + 8 * u, rb = tb * kDcCovTile + r0 + 8 * u;
    ma[u] = ra < M ? mean[ra] : 0.0;
    mb[u] = rb < M ? mean[rb] : 0.0;
  }
  auto load = [&](int64_t n0) {
    const int64_t n = n0 + kk;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int ra = ta * kDcCovTile + r0 + 8 * u, rb = tb * kDcCovTile + r0 + 8 * u;
      xa[u] = ra < M && n < nb1 ? X[(int64_t)ra * N + n] : ma[u];
      xb[u] = rb < M && n < nb1 ? X[(int64_t)rb * N + n] : mb[u];
    }
  };
  load(nb0);
  for (int64_t n0 = nb0; n0 < nb1; n0 += kDcChunk) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      sa[r0 + 8 * u][kk] = xa[u] - ma[u];
      sb[r0 + 8 * u][kk] = xb[u] - mb[u];
    }
    if (n0 + kDcChunk < nb1) load(n0 + kDcChunk);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kDcChunk; k += 4) {
      const double a0 = sa[wa + c][k + g], a1 = sa[wa + 16 + c][k + g];
      const double b0 = sb[wb + c][k + g], b1 = sb[wb + 16 + c][k + g];
      acc[0][0] = mma(a0, b0, acc[0][0]);
      acc[0][1] = mma(a0, b1, acc[0][1]);
      acc[1][0] = mma(a1, b0, acc[1][0]);
      acc[1][1] = mma(a1, b1, acc[1][1]);
    }
  }
  double* out = P + (int64_t)blockIdx.y * M * M;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ra = ta * kDcCovTile + wa + 16 * u + 4 * r + g;
        const int rb = tb * kDcCovTile + wb + 16 * v + c;
        if (ra < M && rb < M) out[(int64_t)ra * M + rb] = acc[u][v][r];
      }
}

// C = sum of the slices' partials (in slice order) / (N - 1), both triangles.
__global__ void __launch_bounds__(256) k_dc_cov_sum(int M, int64_t N, int n_slices,
                                                    const double* __restrict__ P,
                                                    double* __restrict__ Cv) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)M * M) return;
  const int a = (int)(q / M), b = (int)(q % M);
  if (b > a) return;
  double s = 0.0;
  for (int z = 0; z < n_slices; ++z) s += P[(int64_t)z * M * M + q];
  const double v = s / (double)(N - 1);
  Cv[(int64_t)a * M + b] = v;
  Cv[(int64_t)b * M + a] = v;
}

// Cholesky of the M x M matrix A (both triangles; not overwritten) by columns of
// 16x16 tiles, one workgroup.  For block column j a wave forms the tiles
// (ti, j), ti = j + wave, j + wave + 16, ..., of A - sum_k L_k L_k^T on the matrix
// cores, transposed (rows of block j, columns of block ti), and keeps them in LDS; wave 0,
// which has the diagonal tile, factors it (a row per lane) and inverts the factor,
// and the other tiles are multiplied by that inverse: as in the substitution below a
// tile's registers are the operand of that product.  Two barriers per block column
// and no pass over the trailing matrix.  L is written transposed to LT (LT[k][i] =
// L[i][k], the layout the substitution reads), the inverses of its diagonal blocks
// to Di in the order of a matrix A operand (Di[b][s][l]: row l%16, column
// 4 s + l/16).  Bound by the chain of the 16 pivots of each diagonal tile: 300
// rows 546 -> 230 us (before, blocks of 32 columns factored in LDS with four
// barriers per column, and a trailing update on the vector units).
//
// A pivot of at most 1e-12 of its diagonal entry marks a row that is (to rounding) a
// combination of the rows before it: *status is set and LT is made the identity,
// so that the later steps leave the design as it is.
__global__ void __launch_bounds__(kDcCholThreads) k_dc_chol(int M, const double* __restrict__ A,
                                                            double* __restrict__ LT,
                                                            double* __restrict__ Di,
                                                            int32_t* __restrict__ status) {
  extern __shared__ double s_T[];  // the block column's tiles [nt][4][64]: a lane's registers
  __shared__ double s_D[kDcT][kDcT + 1];  // the diagonal tile
  __shared__ double s_Di[kDcT * kDcT];    // the inverse of its factor, operand order
  __shared__ int s_bad;
  const int tid = threadIdx.x, wave = tid / 64, l = tid % 64, c = l & 15, g = l >> 4;
  const int nt = (M + kDcT - 1) / kDcT;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  for (int j = 0; j < nt; ++j) {
    const int ra = kDcT * j + c;  // column of LT of the A operand (row of block j)
    const int la = (ra < M ? ra : 0) + g * M;
#pragma unroll 1
    for (int ti = j + wave; ti < nt; ti += kDcCholThreads / 64) {
      const int rb = kDcT * ti + c;
      const int lb = (rb < M ? rb : 0) + g * M;
      d4v a0, a1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = kDcT * j + 4 * r + g;
        a0[r] = row < M && rb < M ? A[(int64_t)row * M + rb] : 0.0;
      }
#pragma unroll 4
      for (int k = 0; k < j; ++k) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double* row = LT + (kDcT * k + 4 * s) * M;  // (M <= 1024: 32-bit offsets)
          const double va = row[la], vb = row[lb];
          if (s & 1)
            a1 = mma(ra < M ? -va : 0.0, rb < M ? vb : 0.0, a1);
          else
            a0 = mma(ra < M ? -va : 0.0, rb < M ? vb : 0.0, a0);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) s_T[((ti - j) * 4 + r) * 64 + l] = a0[r] + a1[r];
    }
    if (wave == 0) {
      const int nb = std::min(kDcT, M - kDcT * j);
      int c = l & 15;  // opaque: the masks and addresses below are not kept across blocks
      asm volatile("" : "+v"(c));
#pragma unroll
      for (int r = 0; r < 4; ++r) s_D[4 * r + g][c] = s_T[r * 64 + l];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // row c of the tile per lane (each quarter of the wave has all of them); rows
      // past M are the identity
      double a[kDcT];
#pragma unroll
      for (int k = 0; k < kDcT; ++k) a[k] = c < nb && k <= c ? s_D[c][k] : (k == c ? 1.0 : 0.0);
      const double d0 = c < nb ? A[(int64_t)(kDcT * j + c) * M + kDcT * j + c] : 0.0;
      // the inverse by the same row operations on the identity: x[m] = row c, column m
      double x[kDcT];
#pragma unroll
      for (int m = 0; m < kDcT; ++m) x[m] = m == c ? 1.0 : 0.0;
      bool bad = false;
#pragma unroll
      for (int k = 0; k < kDcT; ++k) {
        double d = row_lane(a[k], k);
        if (!(d > 1e-12 * row_lane(d0, k))) {
          bad = true;
          d = 1.0;
        }
        // 1 / sqrt(d) from the hardware estimate and two Newton steps
        double y = __builtin_amdgcn_rsq(d);
        y = y * fma(-0.5 * d * y, y, 1.5);
        y = y * fma(-0.5 * d * y, y, 1.5);
        const double rt = d * y;
        const double lk = c == k ? fma(fma(-rt, rt, d), 0.5 * y, rt) : a[k] * y;
        a[k] = lk;
#pragma unroll
        for (int m = k + 1; m < kDcT; ++m) a[m] = fma(-lk, row_lane(lk, m), a[m]);
#pragma unroll
        for (int m = 0; m <= k; ++m) {
          const double xk = row_lane(x[m], k) * y;
          x[m] = c == k ? xk : (c > k ? fma(-lk, xk, x[m]) : x[m]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (bad && l == 0) s_bad = 1;
      if (g == 0) {  // entry (c, m): step m / 4, lane c + 16 (m % 4)
#pragma unroll
        for (int m = 0; m < kDcT; ++m) {
          const int e = (m >> 2) * 64 + 16 * (m & 3) + c;
          s_Di[e] = x[m];
          Di[(int64_t)j * kDcT * kDcT + e] = x[m];
        }
#pragma unroll
        for (int k = 0; k < kDcT; ++k)
          if (k <= c && c < nb) LT[(int64_t)(kDcT * j + k) * M + kDcT * j + c] = a[k];
      }
    }
    __syncthreads();
    if (s_bad) break;  // uniform: shared flag read after the barrier
#pragma unroll 1
    for (int ti = j + wave; ti < nt; ti += kDcCholThreads / 64) {
      if (ti == j) continue;  // a tile below: block j is whole
      d4v z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s) z = mma(s_Di[s * 64 + l], s_T[((ti - j) * 4 + s) * 64 + l], z);
      const int col = kDcT * ti + c;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (col < M) LT[(int64_t)(kDcT * j + 4 * r + g) * M + col] = z[r];
    }
    __syncthreads();  // the block's columns of LT are complete
  }
  if (s_bad) {
    for (int64_t q = tid; q < (int64_t)M * M; q += kDcCholThreads)
      LT[q] = (q / M == q % M) ? 1.0 : 0.0;
    for (int q = tid; q < nt * kDcT * kDcT; q += kDcCholThreads) {
      const int e = q % (kDcT * kDcT);
      Di[q] = e % 16 == 4 * (e / 64) + e % 64 / 16 ? 1.0 : 0.0;
    }
  }
  if (tid == 0) *status = s_bad;
}

// Z[:, n] = L^{-1} (X[:, n] - mean) by blocks of 16 rows, a wave per 16 samples:
// block b is the residual X_b - mean - sum_k L_bk Z_k on the matrix cores, then the
// product with the inverse of L_bb.  The scores of the wave's samples stay in LDS
// ([M][16]); a lane reads back what it wrote itself (operand layouts, see the top),
// so there is no barrier.  Bound by the reads of L (half of M^2 values per wave,
// from L2) and the chain of matrix operations of a wave: 300 rows of 1e4 samples,
// 625 waves, 496 -> 80 us (a substitution by rows on the vector units before).
__global__ void __launch_bounds__(64) k_dc_whiten(int M, int64_t N, const double* __restrict__ X,
                                                  const double* __restrict__ mean,
                                                  const double* __restrict__ LT,
                                                  const double* __restrict__ Di,
                                                  double* __restrict__ Z) {
  extern __shared__ double s_z[];  // [16 n_blk][16]
  const int l = threadIdx.x, c = l & 15, g = l >> 4;
  const int64_t n = (int64_t)blockIdx.x * kDcT + c;
  const bool ok = n < N;
  const int n_blk = (M + kDcT - 1) / kDcT;
  auto residual = [&](int b, d4v& x) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = kDcT * b + 4 * r + g;
      x[r] = ok && row < M ? X[(int64_t)row * N + n] - mean[row] : 0.0;
    }
  };
  // L comes in batches of four blocks (decor_plan.hpp), the next one's loads (the
  // next row of blocks' first batch at the end of a row) ahead of this one's products;
  // a single block row has nothing to load
  constexpr int kB = kDcBatch;
  auto load = [&](DcBatch t, double (&v)[kB][4]) {
    const int row = kDcT * t.b + c;
    const double* lt = LT + (row < M ? row : 0) + (int64_t)g * M;
#pragma unroll
    for (int q = 0; q < kB; ++q)
#pragma unroll
      for (int s = 0; s < 4; ++s) v[q][s] = lt[(int64_t)dc_row(t.block(q), s, 0) * M];
  };
  d4v next;
  double cur[kB][4], nxt[kB][4];
  residual(0, next);
  if (dc_first_batch().b < n_blk) load(dc_first_batch(), cur);
  for (int b = 0; b < n_blk; ++b) {
    d4v acc = next, acc1 = {0.0, 0.0, 0.0, 0.0};
    if (b + 1 < n_blk) residual(b + 1, next);  // loads ahead of this block's products
    const bool in = kDcT * b + c < M;  // (a row past M read what LT does not hold)
    for (int k0 = 0; k0 < b; k0 += kB) {
      const DcBatch nx = dc_next_batch({b, k0});
      if (nx.b < n_blk) load(nx, nxt);  // uniform
#pragma unroll
      for (int q = 0; q < kB; ++q) {
        if (k0 + q < b) {  // uniform
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const double zv = s_z[(kDcT * (k0 + q) + 4 * s + g) * kDcT + c];
            if (s & 1)
              acc1 = mma(in ? -cur[q][s] : 0.0, zv, acc1);
            else
              acc = mma(in ? -cur[q][s] : 0.0, zv, acc);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < kB; ++q)
#pragma unroll
        for (int s = 0; s < 4; ++s) cur[q][s] = nxt[q][s];
    }
    d4v z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) z = mma(Di[(int64_t)b * 256 + s * 64 + l], acc[s] + acc1[s], z);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int zr = kDcT * b + 4 * r + g;
      s_z[zr * kDcT + c] = z[r];
      if (ok && zr < M) Z[(int64_t)zr * N + n] = z[r];
    }
  }
}

// Total order on the bits of a double (negative values below positive ones,
// -0 taken as +0): the order of the values wherever they are comparable.
__device__ __forceinline__ uint64_t order_key(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v + 0.0);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Ranks of the entries of every row, by buckets: the finite range [lo, hi] of
// a row is cut into N equal buckets (a monotone map, so a lower bucket never
// holds a larger value), bucket offsets come from a prefix sum of the counts,
// and an entry's rank is its bucket's offset plus the entries of its own
// bucket that come before it (smaller key, or equal key and lower index).
// Expected O(N) per row for continuous values.  Non-finite values go to the
// end buckets (NaN to the first), so the ranks stay a permutation whatever
// the values are; the bucket of each entry is computed once and stored, so
// that the count, the placement and the rank see the same bucket.
__global__ void __launch_bounds__(256) k_dc_range(int64_t N, const double* __restrict__ V,
                                                  double2* __restrict__ lohi) {
  const double* v = V + (int64_t)blockIdx.x * N;
  double lo = INFINITY, hi = -INFINITY;
  for (int64_t n = threadIdx.x; n < N; n += 256) {
    const double x = v[n];
    if (isfinite(x)) {
      lo = fmin(lo, x);
      hi = fmax(hi, x);
    }
  }
  __shared__ double s_lo[256], s_hi[256];
  s_lo[threadIdx.x] = lo;
  s_hi[threadIdx.x] = hi;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s_lo[threadIdx.x] = fmin(s_lo[threadIdx.x], s_lo[threadIdx.x + w]);
      s_hi[threadIdx.x] = fmax(s_hi[threadIdx.x], s_hi[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    lo = s_lo[0];
    hi = s_hi[0];
    const double span = hi - lo;
    // scale 0 (one bucket) if the row has no finite spread
    const double scale = (lo <= hi && span > 0.0 && span < INFINITY) ? (double)N / span : 0.0;
    lohi[blockIdx.x] = make_double2(lo <= hi ? lo : 0.0, scale);
  }
}

__global__ void __launch_bounds__(256) k_dc_zero(int64_t count, int32_t* __restrict__ a,
                                                 int32_t* __restrict__ b) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < count) {
    a[q] = 0;
    b[q] = 0;
  }
}

__global__ void __launch_bounds__(256) k_dc_bucket(int64_t N, const double* __restrict__ V,
                                                   const double2* __restrict__ lohi,
                                                   int32_t* __restrict__ bkt,
                                                   int32_t* __restrict__ cnt) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int64_t row = (int64_t)blockIdx.y * N;
  const double2 ls = lohi[blockIdx.y];
  const double f = (V[row + n] - ls.x) * ls.y;
  int32_t b;
  if (!(f >= 0.0))
    b = 0;  // NaN, -inf
  else if (!(f < (double)N))
    b = (int32_t)(N - 1);  // +inf, the top of the range
  else
    b = (int32_t)f;
  bkt[row + n] = b;
  atomicAdd(&cnt[row + b], 1);
}

// Exclusive prefix sum of each row of cnt in place (one workgroup per row).
__global__ void __launch_bounds__(1024) k_dc_scan(int64_t N, int32_t* __restrict__ cnt) {
  int32_t* c = cnt + (int64_t)blockIdx.x * N;
  __shared__ int32_t s[1024];
  int32_t carry = 0;
  for (int64_t c0 = 0; c0 < N; c0 += 1024) {
    const int64_t q = c0 + threadIdx.x;
    const int32_t v = q < N ? c[q] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int w = 1; w < 1024; w <<= 1) {
      const int32_t add = (int)threadIdx.x >= w ? s[threadIdx.x - w] : 0;
      __syncthreads();
      s[threadIdx.x] += add;
      __syncthreads();
    }
    if (q < N) c[q] = carry + s[threadIdx.x] - v;
    carry += s[1023];
    __syncthreads();  // s is rewritten by the next chunk
  }
}

__global__ void __launch_bounds__(256) k_dc_place(int64_t N, const int32_t* __restrict__ bkt,
                                                  const int32_t* __restrict__ off,
                                                  int32_t* __restrict__ fill,
                                                  int32_t* __restrict__ perm) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int64_t row = (int64_t)blockIdx.y * N;
  const int32_t b = bkt[row + n];
  const int32_t slot = off[row + b] + atomicAdd(&fill[row + b], 1);
  perm[row + slot] = (int32_t)n;
}

// R[i][n] = rank (if R), inv[i][rank] = n (if inv).
__global__ void __launch_bounds__(256) k_dc_rank(int64_t N, const double* __restrict__ V,
                                                 const int32_t* __restrict__ bkt,
                                                 const int32_t* __restrict__ off,
                                                 const int32_t* __restrict__ perm,
                                                 int32_t* __restrict__ R,
                                                 int32_t* __restrict__ inv) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int64_t row = (int64_t)blockIdx.y * N;
  const int32_t b = bkt[row + n];
  const int32_t o0 = off[row + b];
  const int32_t o1 = b + 1 < N ? off[row + b + 1] : (int32_t)N;
  const uint64_t key = order_key(V[row + n]);
  int32_t r = o0;
  for (int32_t p = o0; p < o1; ++p) {
    const int32_t m = perm[row + p];
    const uint64_t km = order_key(V[row + m]);
    r += (km < key) || (km == key && m < n);
  }
  if (R) R[row + n] = r;
  if (inv) inv[row + r] = (int32_t)n;
}

// The ranks of a row (as k_dc_range .. k_dc_rank) by one workgroup, counts and
// order in LDS: [N + 1] bucket offsets, [N] entries by bucket and, with VALUES, their
// values (rows up to kDcRowValues; else the values of a bucket's entries are read
// from memory again).  A thread keeps its entries in registers.  The global form's
// counters and orders make six passes with an atomic per entry and pass to L2: 350
// us for 300 rows of 1e4, 48 us here.
//
// Counting inside a bucket is quadratic in its entries.  Where a design has fewer
// rows than the chip has CUs, gridDim.y workgroups form a row's buckets, each for
// itself, and count in a share of them (the share of a bucket follows from its offset,
// which is the same in all).  A row whose counting would still cost more than sorting
// it (an outlier that stretches the range, few distinct values, heavy tails) is
// sorted by the first workgroup: runs of 1, 2, 4, ... entries of the order merge, each
// entry finding its place in the other run by bisection, and the arrays of offsets and
// order take turns.  Whole reduction of 16 rows of 2e4, ms, by one workgroup that counts /
// here / by the global form: normal values 0.22 / 0.15 / 0.36, rounded to 0.05 1.5 / 0.30
// / 0.77, with an outlier 87 / 1.3 / 10; kDcCrowd is where sorting takes over, within a
// tenth of the best from 128 to 300.
template <bool VALUES>
__global__ void __launch_bounds__(kDcRankThreads) k_dc_rank_row(int N, const double* __restrict__ V,
                                                                int32_t* __restrict__ R,
                                                                int32_t* __restrict__ inv) {
  constexpr int64_t kMax = VALUES ? kDcRowValues : kDcRowMax;
  constexpr int kPer = (int)((kMax + kDcRankThreads - 1) / kDcRankThreads);
  extern __shared__ double s_val[];  // with VALUES [N]; then [N + 1] offsets, the order [N]
  int32_t* s_off = reinterpret_cast<int32_t*>(VALUES ? s_val + N : s_val);
  int32_t* s_perm = s_off + N + 1;
  __shared__ double s_lo[kDcRankThreads / 64], s_hi[kDcRankThreads / 64];
  __shared__ int32_t s_sum[kDcRankThreads / 64], s_work[kDcRankThreads / 64];
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  const int64_t row = (int64_t)blockIdx.x * N;
  const double* v = V + row;
  double x[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int n = tid + j * kDcRankThreads;
    x[j] = v[n < N ? n : N - 1];
  }
  double lo = INFINITY, hi = -INFINITY;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (isfinite(x[j])) {
      lo = fmin(lo, x[j]);
      hi = fmax(hi, x[j]);
    }
  }
  for (int w = 32; w > 0; w >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, w, 64));
    hi = fmax(hi, __shfl_xor(hi, w, 64));
  }
  if (lane == 0) {
    s_lo[wave] = lo;
    s_hi[wave] = hi;
  }
  for (int q = tid; q <= N; q += kDcRankThreads) s_off[q] = 0;
  __syncthreads();
  for (int w = 0; w < kDcRankThreads / 64; ++w) {
    lo = fmin(lo, s_lo[w]);
    hi = fmax(hi, s_hi[w]);
  }
  const double span = hi - lo;
  const double scale = (lo <= hi && span > 0.0 && span < INFINITY) ? (double)N / span : 0.0;
  if (!(lo <= hi)) lo = 0.0;
  // The row by merging: R and inv as below.
  auto sort_row = [&]() {
    int32_t *src = s_off, *dst = s_perm;
    auto key = [&](int n) { return order_key(VALUES ? s_val[n] : v[n]); };
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int n = tid + j * kDcRankThreads;
      if (n < N) {
        src[n] = n;
        if constexpr (VALUES) s_val[n] = x[j];
      }
    }
    __syncthreads();
    for (int len = 1; len < N; len *= 2) {
#pragma unroll 4
      for (int j = 0; j < kPer; ++j) {
        const int p = tid + j * kDcRankThreads;
        if (p < N) {
          const int n = src[p];
          const uint64_t k = key(n);
          const int base = p & ~(2 * len - 1);         // of the two runs
          const int other = base + ((p & len) ? 0 : len);  // the one without p
          int lo = min(other, N), hi = min(other + len, N);
          const int o0 = lo;
          while (lo < hi) {  // entries of the other run before mine: by value, then by index
            const int mid = (lo + hi) / 2, m = src[mid];
            const uint64_t km = key(m);
            if (km < k || (km == k && m < n))
              lo = mid + 1;
            else
              hi = mid;
          }
          dst[base + (p & (len - 1)) + (lo - o0)] = n;
        }
      }
      __syncthreads();
      int32_t* t = src;
      src = dst;
      dst = t;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int p = tid + j * kDcRankThreads;
      if (p < N) {
        if (R) R[row + src[p]] = p;
        if (inv) inv[row + p] = src[p];
      }
    }
  };
  auto bucket = [&](double y) {
    const double f = (y - lo) * scale;
    return !(f >= 0.0) ? 0 : !(f < (double)N) ? N - 1 : (int32_t)f;  // NaN, -inf; +inf, top
  };
  int32_t bkt[kPer], slot[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int n = tid + j * kDcRankThreads;
    if (n < N) {
      bkt[j] = bucket(x[j]);
      slot[j] = atomicAdd(&s_off[bkt[j]], 1);
    }
  }
  __syncthreads();
  {  // exclusive prefix sum of the counts: a run of buckets per thread
    const int per = (N + kDcRankThreads - 1) / kDcRankThreads;
    const int q0 = tid * per, q1 = min(N, q0 + per);
    int32_t mine = 0;
    int32_t work = 0;    // comparisons: the sum of the counts' squares (N <= 20000: below 2^31)
    bool crowd = false;  // one bucket costs more than the sort by itself
    for (int q = q0; q < q1; ++q) {
      const int32_t c = s_off[q];
      mine += c;
      work += c * c;
      crowd = crowd || c * c > kDcCrowd * N;
    }
    for (int w = 32; w > 0; w >>= 1) work += __shfl_xor(work, w, 64);
    if (__builtin_amdgcn_ballot_w64(crowd) != 0) work = -1;
    if (lane == 0) s_work[wave] = work;
    __syncthreads();
    work = 0;
    crowd = false;
    for (int w = 0; w < kDcRankThreads / 64; ++w) {
      crowd = crowd || s_work[w] < 0;
      work += s_work[w];
    }
    if (crowd || work / kDcCrowd > N * (int)gridDim.y) {  // uniform
      if (blockIdx.y == 0) sort_row();
      return;
    }
    int32_t up = mine;  // inclusive over the wave
    for (int w = 1; w < 64; w <<= 1) {
      const int32_t o = __shfl_up(up, w, 64);
      if (lane >= w) up += o;
    }
    if (lane == 63) s_sum[wave] = up;
    __syncthreads();
    int32_t o = up - mine;
    for (int w = 0; w < wave; ++w) o += s_sum[w];
    for (int q = q0; q < q1; ++q) {
      const int32_t cq = s_off[q];
      s_off[q] = o;
      o += cq;
    }
    if (tid == 0) s_off[N] = N;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int n = tid + j * kDcRankThreads;
    if (n < N) {
      const int32_t p = s_off[bkt[j]] + slot[j];
      s_perm[p] = n;
      if constexpr (VALUES) s_val[p] = x[j];
    }
  }
  __syncthreads();
  // in the order of the buckets: the lanes of a wave walk the same few of them.  My
  // share: the buckets that start in [lo_p, hi_p)
  const int lo_p = (int)((int64_t)blockIdx.y * N / gridDim.y), hi_p = (int)((int64_t)(blockIdx.y + 1) * N / gridDim.y);
#pragma unroll 1
  for (int p = lo_p + tid; p < N; p += kDcRankThreads) {
    const int32_t n = s_perm[p];
    const double y = VALUES ? s_val[p] : v[n];
    const int32_t b = bucket(y), o0 = s_off[b], o1 = s_off[b + 1];
    if (o0 < lo_p) continue;  // the share before has it
    if (o0 >= hi_p) break;
    const uint64_t key = order_key(y);
    int32_t r = o0;
#pragma unroll 4
    for (int32_t q = o0; q < o1; ++q) {
      const int32_t m = s_perm[q];
      const uint64_t km = order_key(VALUES ? s_val[q] : v[m]);
      r += (km < key) || (km == key && m < n);
    }
    if (R) R[row + n] = r;
    if (inv) inv[row + r] = n;
  }
}

// inv[i][strata[i][n]] = n for a design whose strata are known (an LHS
// design: the order of a row's values is the order of their strata).
__global__ void __launch_bounds__(256) k_dc_invert(int64_t N, const int32_t* __restrict__ strata,
                                                   int32_t* __restrict__ inv) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int64_t row = (int64_t)blockIdx.y * N;
  inv[row + strata[row + n]] = (int32_t)n;
}

// out[i][n] = X[i][inv[i][Rz[i][n]]]: the entry whose row rank equals the
// score rank of (i, n); strata[i][n] = that rank.  After a failed
// factorisation (*status != 0) the design is copied as it is.
__global__ void __launch_bounds__(256) k_dc_apply(int64_t N, const double* __restrict__ X,
                                                  const int32_t* __restrict__ inv,
                                                  const int32_t* __restrict__ Rz,
                                                  const int32_t* __restrict__ status,
                                                  double* __restrict__ out,
                                                  int32_t* __restrict__ strata) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int64_t row = (int64_t)blockIdx.y * N;
  const int32_t r = Rz[row + n];
  out[row + n] = *status ? X[row + n] : X[row + inv[row + r]];
  if (strata) strata[row + n] = r;
}

}  // namespace

namespace {

// Covariance launch: lower-triangle tiles times sample slices, about 1024
// workgroups in all, each slice a multiple of the LDS chunk and at least 256
// samples long.
struct CovPlan {
  unsigned n_tiles;
  int64_t per;
  int n_slices;
  CovPlan(int32_t M, int64_t N) {
    const int t1 = (M + kDcCovTile - 1) / kDcCovTile;
    n_tiles = (unsigned)(t1 * (t1 + 1) / 2);
    const int64_t want = std::max<int64_t>(1, 1024 / (int64_t)n_tiles);
    per = (N + want - 1) / want;
    per = std::max<int64_t>(256, (per + kDcChunk - 1) / kDcChunk * kDcChunk);
    n_slices = (int)((N + per - 1) / per);
  }
};

// Rows that a workgroup ranks in LDS; longer ones take the buffers below.
constexpr bool ranked_in_lds(int64_t N) { return N <= kDcRowMax; }

struct RankBufs {
  double2* lohi;
  int32_t *bkt, *off, *fill, *perm;
};

// Ranks of the rows of V[M][N] (R and/or inv, see k_dc_rank).
void launch_rank(int32_t M, int64_t N, const double* V, const RankBufs& b, int32_t* R,
                 int32_t* inv, hipStream_t st) {
  const size_t words = (size_t)(2 * N + 1) * sizeof(int32_t);
  // workgroups per row: as many as leave each a CU of its own, for rows long enough that
  // counting may weigh
  const unsigned split = N < 4096 ? 1u : (unsigned)std::max(1, std::min(kDcRankSplit, 256 / M));
  if (N <= kDcRowValues) {
    hipLaunchKernelGGL(k_dc_rank_row<true>, dim3((unsigned)M, split), dim3(kDcRankThreads),
                       words + (size_t)N * sizeof(double), st, (int)N, V, R, inv);
    return;
  }
  if (ranked_in_lds(N)) {
    hipLaunchKernelGGL(k_dc_rank_row<false>, dim3((unsigned)M, split), dim3(kDcRankThreads), words, st,
                       (int)N, V, R, inv);
    return;
  }
  const unsigned gs = (unsigned)((N + 255) / 256);
  const int64_t MN = (int64_t)M * N;
  hipLaunchKernelGGL(k_dc_range, dim3((unsigned)M), dim3(256), 0, st, N, V, b.lohi);
  hipLaunchKernelGGL(k_dc_zero, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, st, MN, b.off,
                     b.fill);
  hipLaunchKernelGGL(k_dc_bucket, dim3(gs, (unsigned)M), dim3(256), 0, st, N, V,
                     (const double2*)b.lohi, b.bkt, b.off);
  hipLaunchKernelGGL(k_dc_scan, dim3((unsigned)M), dim3(1024), 0, st, N, b.off);
  hipLaunchKernelGGL(k_dc_place, dim3(gs, (unsigned)M), dim3(256), 0, st, N,
                     (const int32_t*)b.bkt, (const int32_t*)b.off, b.fill, b.perm);
  hipLaunchKernelGGL(k_dc_rank, dim3(gs, (unsigned)M), dim3(256), 0, st, N, V,
                     (const int32_t*)b.bkt, (const int32_t*)b.off, (const int32_t*)b.perm, R, inv);
}

}  // namespace

size_t decorrelate_workspace(int32_t M, int64_t N) {
  const CovPlan cp(M, N);
  return (size_t)M * N * (sizeof(double) + (ranked_in_lds(N) ? 3 : 7) * sizeof(int32_t)) +
         ((size_t)cp.n_slices + 2) * M * M * sizeof(double) + 3 * (size_t)M * sizeof(double2) +
         (size_t)(M + kDcT - 1) / kDcT * 256 * sizeof(double) + 8 * 256;
}

int decorrelate_design(Context* c, int32_t M, int64_t N, double* zeta, int32_t* strata,
                       const int32_t* lhs_strata, int32_t** status_out, hipStream_t st) {
  if (M < 1 || M > kDecorMaxM || N <= M || N > kDecorMaxN)
    return fail(FMC_EINVAL, "correlation reduction needs M <= 1024 and M < N < 2^31");
  const size_t MN = (size_t)M * N;
  const CovPlan cp(M, N);
  void *z, *rz, *inv, *part, *cv, *lt, *di, *mean, *sts;
  void *bkt = nullptr, *off = nullptr, *fill = nullptr, *perm = nullptr, *lohi = nullptr;
  int rc;
  if ((rc = c->ensure("dc_z", MN * sizeof(double), &z))) return rc;
  if ((rc = c->ensure("dc_rz", MN * sizeof(int32_t), &rz))) return rc;
  if ((rc = c->ensure("dc_inv", MN * sizeof(int32_t), &inv))) return rc;
  if (!ranked_in_lds(N)) {
    if ((rc = c->ensure("dc_bkt", MN * sizeof(int32_t), &bkt))) return rc;
    if ((rc = c->ensure("dc_off", MN * sizeof(int32_t), &off))) return rc;
    if ((rc = c->ensure("dc_fill", MN * sizeof(int32_t), &fill))) return rc;
    if ((rc = c->ensure("dc_perm", MN * sizeof(int32_t), &perm))) return rc;
    if ((rc = c->ensure("dc_lohi", (size_t)M * sizeof(double2), &lohi))) return rc;
  }
  if ((rc = c->ensure("dc_part", (size_t)cp.n_slices * M * M * sizeof(double), &part))) return rc;
  if ((rc = c->ensure("dc_c", (size_t)M * M * sizeof(double), &cv))) return rc;
  if ((rc = c->ensure("dc_lt", (size_t)M * M * sizeof(double), &lt))) return rc;
  if ((rc = c->ensure("dc_di", (size_t)(M + kDcT - 1) / kDcT * 256 * sizeof(double), &di))) return rc;
  if ((rc = c->ensure("dc_mean", (size_t)M * sizeof(double), &mean))) return rc;
  if ((rc = c->ensure("dc_status", 256, &sts))) return rc;
  double* Z = (double*)z;
  double* mu = (double*)mean;
  int32_t* status = (int32_t*)sts;
  const RankBufs rb{(double2*)lohi, (int32_t*)bkt, (int32_t*)off, (int32_t*)fill, (int32_t*)perm};
  const unsigned gs = (unsigned)((N + 255) / 256);
  hipLaunchKernelGGL(k_dc_mean, dim3((unsigned)M), dim3(256), 0, st, N, zeta, mu);
  hipLaunchKernelGGL(k_dc_cov, dim3(cp.n_tiles, (unsigned)cp.n_slices), dim3(256), 0, st, M, N,
                     cp.per, zeta, mu, (double*)part);
  hipLaunchKernelGGL(k_dc_cov_sum, dim3((unsigned)(((int64_t)M * M + 255) / 256)), dim3(256), 0, st,
                     M, N, cp.n_slices, (const double*)part, (double*)cv);
  const size_t tiles = (size_t)((M + kDcT - 1) / kDcT) * kDcT * kDcT * sizeof(double);
  hipLaunchKernelGGL(k_dc_chol, dim3(1), dim3(kDcCholThreads), tiles, st, M, (const double*)cv,
                     (double*)lt, (double*)di, status);
  hipLaunchKernelGGL(k_dc_whiten, dim3((unsigned)((N + kDcT - 1) / kDcT)), dim3(64),
                     tiles, st, M, N, zeta, mu, (const double*)lt, (const double*)di, Z);
  launch_rank(M, N, Z, rb, (int32_t*)rz, nullptr, st);
  // the design's own ranks, kept only as their inverse (the entry of each
  // rank); an LHS design's strata are those ranks
  if (lhs_strata)
    hipLaunchKernelGGL(k_dc_invert, dim3(gs, (unsigned)M), dim3(256), 0, st, N, lhs_strata,
                       (int32_t*)inv);
  else
    launch_rank(M, N, zeta, rb, nullptr, (int32_t*)inv, st);
  // Z is free once its ranks are taken: it receives the rearranged design
  hipLaunchKernelGGL(k_dc_apply, dim3(gs, (unsigned)M), dim3(256), 0, st, N, zeta,
                     (const int32_t*)inv, (const int32_t*)rz, (const int32_t*)status, Z, strata);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess)
    e = hipMemcpyAsync(zeta, Z, MN * sizeof(double), hipMemcpyDeviceToDevice, st);
  if (e != hipSuccess) return fail(FMC_EDEVICE, hipGetErrorString(e));
  if (status_out) *status_out = status;
  return FMC_OK;
}

}  // namespace fmc
