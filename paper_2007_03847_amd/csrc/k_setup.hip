// k_setup.hip -- scenario setup on the GPU (FP64): Kron reduction of the
// network equations, operating point, packed coefficients; and the ordered
// cross-sample merge of the per-group statistics.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fmc_internal.hpp"

namespace fmc {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
  // Smith's algorithm
  if (fabs(b.x) >= fabs(b.y)) {
    const double r = b.y / b.x, d = b.x + b.y * r;
    return make_double2((a.x + a.y * r) / d, (a.y - a.x * r) / d);
  }
  const double r = b.x / b.y, d = b.x * r + b.y;
  return make_double2((a.x * r + a.y) / d, (a.y * r - a.x) / d);
}

// Quotients by one b, as cdiv (Smith's algorithm): what depends on b alone is formed
// once, and the three divisions are a reciprocal (the hardware's estimate and two
// Newton steps) with the quotient corrected by its residual, which gives a / b = -1
// exactly where a = -b, as a division does, at half its latency.  These divisions are
// on the chain of every elimination step.
struct Divisor {
  double r, d, y;  // ratio of b's parts, Smith's denominator and its reciprocal
  bool re;         // |Re b| >= |Im b|
};
__device__ __forceinline__ double recip(double b) {
  double y = __builtin_amdgcn_rcp(b);
  y = fma(fma(-b, y, 1.0), y, y);
  return fma(fma(-b, y, 1.0), y, y);
}
__device__ __forceinline__ double quot(double a, double b, double y) {
  const double q = a * y;
  return fma(fma(-b, q, a), y, q);
}
__device__ __forceinline__ Divisor divisor(double2 b) {
  Divisor v;
  v.re = fabs(b.x) >= fabs(b.y);
  const double hi = v.re ? b.x : b.y, lo = v.re ? b.y : b.x;
  v.r = quot(lo, hi, recip(hi));
  v.d = hi + lo * v.r;
  v.y = recip(v.d);
  return v;
}
__device__ __forceinline__ double2 quotient(double2 a, const Divisor& v) {
  const double re = v.re ? a.x + a.y * v.r : a.x * v.r + a.y;
  const double im = v.re ? a.y - a.x * v.r : a.y * v.r - a.x;
  return make_double2(quot(re, v.d, v.y), quot(im, v.d, v.y));
}

// ---------------------------------------------------------------------------
// Kron reduction (eq. 2 eliminated) of a small network: one workgroup of 512
// threads, bound by the latency of its n_bus elimination steps.  The augmented
// system [Y_BB | Y_BA] (n_bus rows, W = n_bus + n_gen columns) lives in LDS when
// it fits (n_bus W <= 4096).  Branches, loads and generators enter a row in
// index order, so the sums are deterministic.  Gauss-Jordan elimination with
// partial pivoting on rows that stay where they are: in step k every wave
// finds the pivot (the largest max(|Re|, |Im|) of a_rk, to 14 bits, over the rows
// not yet used, the lowest row on ties) by itself, and every element of the other rows and of the columns
// beyond k is updated from the pivot row and column k, which the step leaves
// alone, so one barrier per step suffices and no back substitution follows:
// X = Y_BB^-1 Y_BA stands in the pivot rows and Y_red = Y_AA - Y_AB X.  39 buses
// and 10 machines: 160 us with row exchanges, four barriers per step, a
// complex division per element and a back substitution; 49 us here.
//
// The pivot row is divided by the pivot, not multiplied by its reciprocal: of two
// buses that only a line joins, the quotient is -1 and the second pivot cancels to
// zero, so that such a network is refused; and the quotient of admittances of any
// size stays in range.
// ---------------------------------------------------------------------------
constexpr int kKronLdsComplex = 4096;  // 64 KB of double2
constexpr int kKronStage = 256;        // branches staged in LDS at a time

// The largest key over the wave's lanes: rows of 16 by DPP, then the four rows.
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
  auto step = [&](unsigned o) { v = o > v ? o : v; };
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // lane ^ 1
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // lane ^ 2
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // half row mirrored
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // row mirrored
  const unsigned r0 = __builtin_amdgcn_readlane((int)v, 0), r1 = __builtin_amdgcn_readlane((int)v, 16),
                 r2 = __builtin_amdgcn_readlane((int)v, 32), r3 = __builtin_amdgcn_readlane((int)v, 48);
  const unsigned a = r0 > r1 ? r0 : r1, b = r2 > r3 ? r2 : r3;
  return a > b ? a : b;
}

__global__ void __launch_bounds__(512) k_kron(NetDev net, double2* __restrict__ Yred, int* status) {
  const int nb = net.n_bus, ng = net.n_gen, W = nb + ng;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
  __shared__ double2 A[kKronLdsComplex];
  __shared__ int s_from[kKronStage], s_to[kKronStage];
  __shared__ double2 s_y[kKronStage];
  __shared__ double s_sh[kKronStage];
  for (int q = tid; q < nb * W; q += nt) A[q] = make_double2(0.0, 0.0);
  // assembly: thread b owns row b; the branches' data is staged by all
  for (int k0 = 0; k0 < net.n_branch; k0 += kKronStage) {
    const int m = net.n_branch - k0 < kKronStage ? net.n_branch - k0 : kKronStage;
    __syncthreads();
    for (int k = tid; k < m; k += nt) {
      s_from[k] = net.from[k0 + k];
      s_to[k] = net.to[k0 + k];
      s_y[k] = cdiv(make_double2(1.0, 0.0), make_double2(net.r[k0 + k], net.x[k0 + k]));
      s_sh[k] = net.b ? 0.5 * net.b[k0 + k] : 0.0;
    }
    __syncthreads();
    for (int b = tid; b < nb; b += nt) {
      double2* row = A + b * W;
#pragma unroll 4
      for (int k = 0; k < m; ++k) {
        const int f = s_from[k], t = s_to[k];
        if (f != b && t != b) continue;
        row[b] = cadd(row[b], cadd(s_y[k], make_double2(0.0, s_sh[k])));
        const int o = (f == b) ? t : f;
        row[o] = csub(row[o], s_y[k]);
      }
    }
  }
  __syncthreads();
  for (int g = tid; g < ng && g < kKronStage; g += nt) s_from[g] = net.gen_bus[g];
  __syncthreads();
  for (int b = tid; b < nb; b += nt) {
    double2* row = A + b * W;
    row[b] = cadd(row[b], make_double2(net.lg ? net.lg[b] : 0.0, net.lb ? net.lb[b] : 0.0));
    for (int g = 0; g < ng; ++g) {  // machines in index order
      const int gb = g < kKronStage ? s_from[g] : net.gen_bus[g];
      if (gb != b) continue;
      const double2 yg = make_double2(0.0, -1.0 / net.xdp[g]);  // 1/(j X'd)
      row[b] = cadd(row[b], yg);
      row[nb + g] = csub(row[nb + g], yg);  // Y_BA = -yg
    }
  }
  __syncthreads();
  // n_bus (n_bus + n_gen) <= 4096 means at most 63 buses: a lane per row
  bool used = lane >= nb;    // row `lane` has been a pivot row (each wave's own copy)
  __shared__ int s_prow[64];  // pivot row and pivot of column k
  __shared__ double2 s_piv[64];
  for (int k = 0; k < nb; ++k) {
    unsigned key = 0;
    if (!used) {
      // exponent and leading bits of the double; |a|^2 that underflows counts as zero
      const double2 v = A[lane * W + k];
      const unsigned m = (unsigned)__double2hiint(fmax(fabs(v.x), fabs(v.y))) & ~63u;
      if (fma(v.x, v.x, v.y * v.y) > 0.0) key = (m > 64u ? m : 64u) | (unsigned)(63 - lane);
    }
    key = wave_max_u32(key);
    if (key == 0) {  // uniform: every wave saw the same column
      if (tid == 0) *status = -1;
      return;
    }
    const int p = 63 - (int)(key & 63u);
    used |= p == lane;
    const double2 akk = A[p * W + k];
    const Divisor by = divisor(akk);
    if (tid == 0) {
      s_prow[k] = p;
      s_piv[k] = akk;
    }
    // a thread takes a column and every 16th row (at most four)
    for (int c = k + 1 + tid % 32; c < W; c += 32) {
      const double2 pc = quotient(A[p * W + c], by);
      double fr[4], fi[4], vr[4], vi[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = tid / 32 + 16 * u, rr = r < nb ? r : p;
        const double2 f = A[rr * W + k], v = A[rr * W + c];
        fr[u] = f.x; fi[u] = f.y; vr[u] = v.x; vi[u] = v.y;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = tid / 32 + 16 * u;
        if (r < nb && r != p)
          A[r * W + c] = make_double2(vr[u] - (fr[u] * pc.x - fi[u] * pc.y), vi[u] - (fr[u] * pc.y + fi[u] * pc.x));
      }
    }
    __syncthreads();
  }
  for (int q = tid; q < ng * ng; q += nt) {
    const int i = q / ng, g = q % ng, b = net.gen_bus[i];
    const double2 yg = make_double2(0.0, -1.0 / net.xdp[i]);
    double2 v = (i == g) ? yg : make_double2(0.0, 0.0);
    const double2 x = cdiv(A[s_prow[b] * W + nb + g], s_piv[b]);
    v = cadd(v, cmul(yg, x));  // -(Y_AB X), Y_AB = -yg
    Yred[q] = v;
  }
  if (tid == 0) *status = 0;
}

// ---------------------------------------------------------------------------
// Large networks (the augmented system does not fit LDS): Kron's node
// elimination on the full admittance matrix of the buses and the generator
// internal nodes (W = n_bus + n_gen, buses first), kKronBlk buses at a time:
// with D the block's diagonal part, Y_ij -= Y_ik D^-1 Y_kj for all remaining i, j,
// formed as (D^-1 S) (S^-1 Y_kj) with S the diagonal of D, so that both factors are
// quotients of admittances (in range whatever their size, and exact for a bus that
// one line joins to the rest: see the singular networks above).
// After the last bus the generator block is Y_red.  The buses are eliminated in
// index order without pivoting: the bus block of a network admittance matrix
// whose series branches share one R/X ratio and whose shunts are loads and
// transient reactances is diagonally dominant.  A zero pivot sets the status.
//
// Bound by the chain of blocks: one launch per block, in which every
// workgroup forms (D^-1 S) (S^-1 Y_kj) of its 64 columns (again in each tile: cheaper than
// another launch) and updates a tile of 32 x 64, and the workgroup of the next
// block's diagonal part forms its D^-1 S before it ends.  780 buses and 200
// machines: 3.9 ms with a launch per bus (780 launches of 4.6 us).
// ---------------------------------------------------------------------------
constexpr int kKronBlk = 32;   // buses per elimination block = rows of a tile
constexpr int kKronCols = 64;  // columns of a tile

// One wave per row: the lanes scan 64 branches (machines) at once, the first
// lane adds the matching ones in index order.
__global__ void __launch_bounds__(64) k_kron_assemble(NetDev net, double2* __restrict__ A,
                                                      int* status) {
  const int nb = net.n_bus, ng = net.n_gen, W = nb + ng;
  const int r = blockIdx.x, lane = threadIdx.x;
  if (r == 0 && lane == 0) *status = 0;  // the elimination steps only ever set -1
  double2* row = A + (int64_t)r * W;      // zeroed before the launch
  if (r >= nb) {
    if (lane == 0) {
      const int g = r - nb;
      const double2 yg = make_double2(0.0, -1.0 / net.xdp[g]);  // 1/(j X'd)
      row[r] = yg;
      row[net.gen_bus[g]] = make_double2(-yg.x, -yg.y);
    }
    return;
  }
  double2 diag = make_double2(0.0, 0.0);
  for (int k0 = 0; k0 < net.n_branch; k0 += 64) {
    const int k = k0 + lane;
    const bool hit = k < net.n_branch && (net.from[k] == r || net.to[k] == r);
    unsigned long long m = __builtin_amdgcn_ballot_w64(hit);
    while (m) {
      const int kk = k0 + __builtin_ctzll(m);
      m &= m - 1;
      if (lane != 0) continue;
      const int f = net.from[kk], t = net.to[kk];
      const double2 y = cdiv(make_double2(1.0, 0.0), make_double2(net.r[kk], net.x[kk]));
      diag = cadd(diag, cadd(y, make_double2(0.0, net.b ? 0.5 * net.b[kk] : 0.0)));
      const int o = (f == r) ? t : f;
      row[o] = csub(row[o], y);
    }
  }
  diag = cadd(diag, make_double2(net.lg ? net.lg[r] : 0.0, net.lb ? net.lb[r] : 0.0));
  for (int g0 = 0; g0 < ng; g0 += 64) {
    const int g = g0 + lane;
    unsigned long long m = __builtin_amdgcn_ballot_w64(g < ng && net.gen_bus[g] == r);
    while (m) {
      const int gg = g0 + __builtin_ctzll(m);
      m &= m - 1;
      if (lane != 0) continue;
      const double2 yg = make_double2(0.0, -1.0 / net.xdp[gg]);
      diag = cadd(diag, yg);
      row[nb + gg] = csub(row[nb + gg], yg);
    }
  }
  if (lane == 0) row[r] = diag;
}

// The scale S of a bus: its diagonal entry, or 1 where that is zero.
__device__ __forceinline__ double2 kron_scale(double2 d) {
  return d.x != 0.0 || d.y != 0.0 ? d : make_double2(1.0, 0.0);
}

// D^-1 S of a kKronBlk x kKronBlk block D by Gauss-Jordan without pivoting, 256
// threads: thread t holds the entries (t / 8, t % 8 + 8 u), u = 0..3; the pivot row
// and column of the next step pass through LDS (two buffers, one barrier per
// step).  Entries past the block's kb rows are the identity's.
struct KronInvLds {
  double2 row[2][kKronBlk], col[2][kKronBlk], scale[kKronBlk];
};
__device__ __forceinline__ void kron_invert(double (&vr)[4], double (&vi)[4], int kb, KronInvLds& s,
                                            int* status) {
  const int i = threadIdx.x / 8, jb = threadIdx.x % 8;
  auto publish = [&](int k) {
    if (i == k) {
#pragma unroll
      for (int u = 0; u < 4; ++u) s.row[k & 1][jb + 8 * u] = make_double2(vr[u], vi[u]);
    }
    if (jb == k % 8) {
      const int h = k / 8;
      const double r = h == 0 ? vr[0] : h == 1 ? vr[1] : h == 2 ? vr[2] : vr[3];
      const double m = h == 0 ? vi[0] : h == 1 ? vi[1] : h == 2 ? vi[2] : vi[3];
      s.col[k & 1][i] = make_double2(r, m);
    }
  };
  publish(0);
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (jb + 8 * u == i) s.scale[i] = kron_scale(make_double2(vr[u], vi[u]));
  __syncthreads();
  for (int k = 0; k < kb; ++k) {
    const double2 piv = s.row[k & 1][k], cik = s.col[k & 1][i], sk = s.scale[k];
    if (!(piv.x != 0.0 || piv.y != 0.0) && threadIdx.x == 0) *status = -1;
    // 1 / a_kk in the pivot row, else -a_ik / a_kk; column k holds the inverse's, times s_k
    const double2 f = quotient(i == k ? make_double2(1.0, 0.0) : make_double2(-cik.x, -cik.y), divisor(piv));
    double2 fs = cmul(f, sk);
    if (i == k && piv.x == sk.x && piv.y == sk.y) fs = make_double2(1.0, 0.0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = jb + 8 * u;
      const double2 akj = s.row[k & 1][j];
      const double2 p = cmul(f, akj);
      const double br = i == k ? 0.0 : vr[u], bi = i == k ? 0.0 : vi[u];
      vr[u] = j == k ? fs.x : br + p.x;
      vi[u] = j == k ? fs.y : bi + p.y;
    }
    if (k + 1 < kb) publish(k + 1);
    __syncthreads();
  }
}

// D^-1 S of the first block (kb = its buses).
__global__ void __launch_bounds__(256) k_kron_first(const double2* __restrict__ A, int W, int kb,
                                                    double2* __restrict__ dinv, int* status) {
  __shared__ KronInvLds s;
  const int i = threadIdx.x / 8, jb = threadIdx.x % 8;
  double vr[4], vi[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = jb + 8 * u;
    const bool on = i < kb && j < kb;
    vr[u] = on ? A[(int64_t)i * W + j].x : (i == j ? 1.0 : 0.0);
    vi[u] = on ? A[(int64_t)i * W + j].y : 0.0;
  }
  kron_invert(vr, vi, kb, s, status);
#pragma unroll
  for (int u = 0; u < 4; ++u) dinv[i * kKronBlk + jb + 8 * u] = make_double2(vr[u], vi[u]);
}

// Elimination of the kb buses k0..k0 + kb - 1: tile (blockIdx.y, blockIdx.x) of
// the trailing matrix (from row and column k1 = k0 + kb on).  dinv: the block's
// D^-1 S; dnext: receives the next block's (nbn buses, 0 after the last).
__global__ void __launch_bounds__(256) k_kron_block(double2* __restrict__ A, int W, int k0, int kb,
                                                    int nbn, const double2* __restrict__ dinv,
                                                    double2* __restrict__ dnext, int* status) {
  __shared__ double2 s_d[kKronBlk][kKronBlk];   // D^-1 S
  __shared__ double2 s_t[kKronBlk][kKronCols];  // S^-1 Y_kj of the tile's columns, then D^-1 Y_kj
  __shared__ double2 s_l[kKronBlk][kKronBlk];   // Y_ik of the tile's rows
  __shared__ KronInvLds s_inv;
  const int tid = threadIdx.x, k1 = k0 + kb;
  const int c0 = k1 + blockIdx.x * kKronCols, r0 = k1 + blockIdx.y * kKronBlk;
  const double2 zero = make_double2(0.0, 0.0);
  for (int q = tid; q < kKronBlk * kKronBlk; q += 256) {
    const int i = q / kKronBlk, j = q % kKronBlk;
    s_d[i][j] = dinv[q];
    s_l[i][j] = (r0 + i < W && j < kb) ? A[(int64_t)(r0 + i) * W + k0 + j] : zero;
  }
  for (int q = tid; q < kKronBlk * kKronCols; q += 256) {
    const int i = q / kKronCols, j = q % kKronCols;
    s_t[i][j] = (i < kb && c0 + j < W) ? quotient(A[(int64_t)(k0 + i) * W + c0 + j],
                                                  divisor(kron_scale(A[(int64_t)(k0 + i) * W + k0 + i])))
                                       : zero;
  }
  __syncthreads();
  // thread: columns tx and tx + 32, rows 4 ty .. 4 ty + 3 of the tile
  const int tx = tid % 32, ty = tid / 32;
  double cr[4][2], ci[4][2];
  auto product = [&](const double2 (*L)[kKronBlk]) {
#pragma unroll
    for (int a = 0; a < 4; ++a) cr[a][0] = cr[a][1] = ci[a][0] = ci[a][1] = 0.0;
#pragma unroll 4
    for (int k = 0; k < kKronBlk; ++k) {
      const double2 x0 = s_t[k][tx], x1 = s_t[k][tx + 32];
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const double2 l = L[4 * ty + a][k];
        cr[a][0] = fma(l.x, x0.x, cr[a][0]);
        cr[a][0] = fma(-l.y, x0.y, cr[a][0]);
        ci[a][0] = fma(l.x, x0.y, ci[a][0]);
        ci[a][0] = fma(l.y, x0.x, ci[a][0]);
        cr[a][1] = fma(l.x, x1.x, cr[a][1]);
        cr[a][1] = fma(-l.y, x1.y, cr[a][1]);
        ci[a][1] = fma(l.x, x1.y, ci[a][1]);
        ci[a][1] = fma(l.y, x1.x, ci[a][1]);
      }
    }
  };
  product(s_d);
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    s_t[4 * ty + a][tx] = make_double2(cr[a][0], ci[a][0]);
    s_t[4 * ty + a][tx + 32] = make_double2(cr[a][1], ci[a][1]);
  }
  __syncthreads();
  product(s_l);
  const bool inverts = nbn > 0 && blockIdx.x == 0 && blockIdx.y == 0;  // uniform
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = r0 + 4 * ty + a, c = c0 + tx + 32 * h;
      double2 v = zero;
      if (r < W && c < W) {
        v = csub(A[(int64_t)r * W + c], make_double2(cr[a][h], ci[a][h]));
        A[(int64_t)r * W + c] = v;
      }
      if (inverts && h == 0) s_d[4 * ty + a][tx] = v;  // read before the last barrier only
    }
  if (!inverts) return;
  __syncthreads();
  const int i = tid / 8, jb = tid % 8;
  double vr[4], vi[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = jb + 8 * u;
    const bool on = i < nbn && j < nbn;
    vr[u] = on ? s_d[i][j].x : (i == j ? 1.0 : 0.0);
    vi[u] = on ? s_d[i][j].y : 0.0;
  }
  kron_invert(vr, vi, nbn, s_inv, status);
#pragma unroll
  for (int u = 0; u < 4; ++u) dnext[i * kKronBlk + jb + 8 * u] = make_double2(vr[u], vi[u]);
}

__global__ void __launch_bounds__(256) k_kron_extract(const double2* __restrict__ A, int nb, int ng,
                                                      double2* __restrict__ Yred) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= ng * ng) return;
  const int W = nb + ng, i = q / ng, k = q % ng;
  Yred[q] = A[(int64_t)(nb + i) * W + nb + k];
}

// The work matrix, then D^-1 S of two diagonal blocks (in turn).
size_t kron_work_bytes(int n_bus, int n_gen) {
  const size_t W = (size_t)n_bus + n_gen;
  return (W * W + 2 * kKronBlk * kKronBlk) * sizeof(double2);
}

hipError_t launch_kron(const NetDev& net, double2* work, double2* Yred, int* status,
                       hipStream_t st) {
  const int nb = net.n_bus, ng = net.n_gen, W = nb + ng;
  if ((int64_t)nb * W <= kKronLdsComplex) {
    hipLaunchKernelGGL(k_kron, dim3(1), dim3(512), 0, st, net, Yred, status);
    return hipGetLastError();
  }
  hipError_t e = launch_fill_i64((int64_t*)work, 0, (int64_t)W * W * 2, st);
  if (e != hipSuccess) return e;
  double2* dinv[2] = {work + (int64_t)W * W, work + (int64_t)W * W + kKronBlk * kKronBlk};
  hipLaunchKernelGGL(k_kron_assemble, dim3((unsigned)W), dim3(64), 0, st, net, work, status);
  hipLaunchKernelGGL(k_kron_first, dim3(1), dim3(256), 0, st, work, W, std::min(kKronBlk, nb),
                     dinv[0], status);
  for (int k0 = 0, q = 0; k0 < nb; k0 += kKronBlk, q ^= 1) {
    const int kb = std::min(kKronBlk, nb - k0), k1 = k0 + kb, m = W - k1;
    const dim3 grid((unsigned)((m + kKronCols - 1) / kKronCols), (unsigned)((m + kKronBlk - 1) / kKronBlk));
    hipLaunchKernelGGL(k_kron_block, grid, dim3(256), 0, st, work, W, k0, kb,
                       std::min(kKronBlk, nb - k1), dinv[q], dinv[q ^ 1], status);
  }
  hipLaunchKernelGGL(k_kron_extract, dim3((unsigned)((ng * ng + 255) / 256)), dim3(256), 0, st,
                     work, nb, ng, Yred);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Operating point.  Pe_i = Re{E~_i conj(I_i)}, I = Y E~ + Yinf V_inf.  Given
// delta0: Pm defaults to Pe(delta0) (equilibrium).  Without delta0 (infinite
// bus): Newton on Pe(delta) = Pm from delta = 0, dense LU with partial
// pivoting.
// ---------------------------------------------------------------------------
// Et and I of the machines at angles d: thread i takes machine i, its current
// summed over k in index order.
__device__ void op_currents(const SetupDev& s, const double* d, double2* Et, double2* I) {
  const int n = s.n;
  for (int k = threadIdx.x; k < n; k += blockDim.x)
    Et[k] = make_double2(s.E[k] * cos(d[k]), s.E[k] * sin(d[k]));
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    double2 c = (s.inf_bus && s.Yinf) ? make_double2(s.Yinf[i].x * s.V_inf, s.Yinf[i].y * s.V_inf)
                                      : make_double2(0.0, 0.0);
#pragma unroll 8
    for (int k = 0; k < n; ++k) c = cadd(c, cmul(s.Y[(int64_t)i * n + k], Et[k]));
    I[i] = c;
  }
  __syncthreads();
}

// One workgroup.  Bound by latency: a thread per machine walks its row of Y
// (one thread for all machines took 47 us for 10 machines and 13.5 ms for
// 200).  The dense solve of a Newton step stays with one thread: an
// infinite-bus system that gives Pm has few machines.
__global__ void __launch_bounds__(256) k_setup(SetupDev s) {
  const int n = s.n, P = s.P, tid = threadIdx.x, bd = blockDim.x;
  CanonLayout L{n, P};
  double* cn = s.canon;
  double* d = cn + L.delta0();
  double2* Et = (double2*)s.work;
  double2* I = Et + n;
  double* J = (double*)(I + n);
  double* rhs = J + (int64_t)n * n;
  __shared__ int s_state;  // 0: iterate, 1: converged, 2: singular
  int ok = 1;
  for (int i = tid; i < n; i += bd) d[i] = s.delta0 ? s.delta0[i] : 0.0;
  if (tid == 0) s_state = 0;
  __syncthreads();
  if (!s.delta0) {
    ok = 0;
    for (int it = 0; it < 100; ++it) {
      op_currents(s, d, Et, I);
      for (int i = tid; i < n; i += bd) {
        const double pe = Et[i].x * I[i].x + Et[i].y * I[i].y;
        rhs[i] = s.Pm[i] - pe;
        for (int k = 0; k < n; ++k) {
          // d Pe_i / d delta_k
          const double2 yk = cmul(s.Y[(int64_t)i * n + k], make_double2(-Et[k].y, Et[k].x));
          double v = Et[i].x * yk.x + Et[i].y * yk.y;
          if (k == i) v += -Et[i].y * I[i].x + Et[i].x * I[i].y;
          J[(int64_t)i * n + k] = v;
        }
      }
      __syncthreads();
      if (tid == 0) {  // solve J dx = rhs
        int sing = 0;
        for (int k = 0; k < n && !sing; ++k) {
          int piv = k;
          double best = fabs(J[(int64_t)k * n + k]);
          for (int r = k + 1; r < n; ++r)
            if (fabs(J[(int64_t)r * n + k]) > best) { best = fabs(J[(int64_t)r * n + k]); piv = r; }
          if (best == 0.0) { sing = 1; break; }
          if (piv != k) {
            for (int c = 0; c < n; ++c) {
              const double t = J[(int64_t)k * n + c];
              J[(int64_t)k * n + c] = J[(int64_t)piv * n + c];
              J[(int64_t)piv * n + c] = t;
            }
            const double t = rhs[k]; rhs[k] = rhs[piv]; rhs[piv] = t;
          }
          for (int r = k + 1; r < n; ++r) {
            const double f = J[(int64_t)r * n + k] / J[(int64_t)k * n + k];
            for (int c = k; c < n; ++c) J[(int64_t)r * n + c] -= f * J[(int64_t)k * n + c];
            rhs[r] -= f * rhs[k];
          }
        }
        if (sing) {
          s_state = 2;
        } else {
          double nrm = 0.0;
          for (int k = n - 1; k >= 0; --k) {
            double acc = rhs[k];
            for (int j = k + 1; j < n; ++j) acc -= J[(int64_t)k * n + j] * rhs[j];
            rhs[k] = acc / J[(int64_t)k * n + k];
          }
          for (int i = 0; i < n; ++i) {
            d[i] += rhs[i];
            nrm = fmax(nrm, fabs(rhs[i]));
          }
          if (nrm <= 1e-15) s_state = 1;
        }
      }
      __syncthreads();
      if (s_state != 0) break;  // uniform: read after the barrier, written before it
    }
    ok = s_state == 1;
  }
  op_currents(s, d, Et, I);
  for (int i = tid; i < n; i += bd) {
    const double pe = Et[i].x * I[i].x + Et[i].y * I[i].y;
    const double pm = s.Pm ? s.Pm[i] : pe;
    cn[L.c0() + i] = Et[i].x;
    cn[L.s0() + i] = Et[i].y;
    cn[L.i0r() + i] = I[i].x;
    cn[L.i0i() + i] = I[i].y;
    cn[L.res() + i] = pm - pe;
    cn[L.dmp() + i] = s.D[i];
    cn[L.inv2h() + i] = 1.0 / (2.0 * s.H[i]);
    cn[L.pm() + i] = pm;
  }
  for (int64_t q = tid; q < (int64_t)n * n; q += bd) {
    cn[L.yre() + q] = s.Y[q].x;
    cn[L.yim() + q] = s.Y[q].y;
  }
  for (int p = tid; p < P; p += bd) {
    cn[L.theta() + p] = s.theta[p];
    cn[L.sigma() + p] = s.sigma[p];
    cn[L.xi0() + p] = s.xi0 ? s.xi0[p] : 0.0;
  }
  if (tid == 0) *s.status = ok ? 0 : -6;
}

hipError_t launch_setup(const SetupDev& s, hipStream_t st) {
  hipLaunchKernelGGL(k_setup, dim3(1), dim3(s.n <= 64 ? 64 : 256), 0, st, s);
  return hipGetLastError();
}

// Coefficients after a network event: the pre-event operating point (E~0,
// D, H, Pm, delta0, the processes) with the post-event admittance: I0 = Yp E~0
// + Yinf V_inf, res = Pm - Re(E~0 conj I0).  A tripped machine keeps no EMF,
// current, mechanical power or residual, so it neither drives nor sees the
// network (its row and column of Yp are zero) and only its damping acts.
__global__ void __launch_bounds__(256) k_setup_post(const double* __restrict__ pre, int n, int P,
                                                    const double2* __restrict__ Yp,
                                                    const double2* __restrict__ Yinf,
                                                    double V_inf, int tripped,
                                                    double* __restrict__ post) {
  const CanonLayout L{n, P};
  const int tid = threadIdx.x, bd = blockDim.x;
  for (int64_t q = tid; q < L.size(); q += bd) post[q] = pre[q];
  __syncthreads();
  for (int64_t q = tid; q < (int64_t)n * n; q += bd) {
    post[L.yre() + q] = Yp[q].x;
    post[L.yim() + q] = Yp[q].y;
  }
  for (int i = tid; i < n; i += bd) {
    double2 I = Yinf ? make_double2(Yinf[i].x * V_inf, Yinf[i].y * V_inf) : make_double2(0.0, 0.0);
    for (int k = 0; k < n; ++k)
      I = cadd(I, cmul(Yp[(int64_t)i * n + k], make_double2(pre[L.c0() + k], pre[L.s0() + k])));
    const double er = pre[L.c0() + i], ei = pre[L.s0() + i];
    const bool out = i == tripped;
    const double pm = out ? 0.0 : pre[L.pm() + i];
    const double pe = out ? 0.0 : er * I.x + ei * I.y;
    post[L.c0() + i] = out ? 0.0 : er;
    post[L.s0() + i] = out ? 0.0 : ei;
    post[L.i0r() + i] = out ? 0.0 : I.x;
    post[L.i0i() + i] = out ? 0.0 : I.y;
    post[L.res() + i] = pm - pe;
    post[L.pm() + i] = pm;
  }
}

hipError_t launch_setup_post(const double* pre, int n, int P, const double2* Yp,
                             const double2* Yinf, double V_inf, int tripped, double* post,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_setup_post, dim3(1), dim3(256), 0, st, pre, n, P, Yp, Yinf, V_inf, tripped,
                     post);
  return hipGetLastError();
}

// Packed, padded coefficients of a variant in its arithmetic type (PackLayout).
template <typename R>
__global__ void __launch_bounds__(256) k_pack(const double* __restrict__ cn, int n, int P,
                                              const int32_t* __restrict__ gen,
                                              const int32_t* __restrict__ owner, bool rotated,
                                              int NG, int PM, R* __restrict__ coef) {
  CanonLayout C{n, P};
  PackLayout L{NG, PM};
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= L.size()) return;
  auto emf = [&](int i) { return make_double2(cn[C.c0() + i], cn[C.s0() + i]); };
  auto conj_emf = [&](int i) { return make_double2(cn[C.c0() + i], -cn[C.s0() + i]); };
  auto scale = [&](int i) { return rotated ? cn[C.inv2h() + i] : 1.0; };
  double v = 0.0;
  if (q < L.binc()) {
    const int e = q < L.yim() ? q : q - L.yim(), i = e / NG, k = e % NG;
    if (i < n && k < n) {
      double2 y = make_double2(cn[C.yre() + (int64_t)i * n + k], cn[C.yim() + (int64_t)i * n + k]);
      if (rotated) y = cmul(cmul(conj_emf(i), y), emf(k));
      v = (q < L.yim() ? y.x : y.y) * scale(i);
    }
  } else if (q < L.c0()) {
    const int e = q - L.binc(), i = e / PM, p = e % PM;
    v = (i < n && p < P && gen[p] == i) ? scale(i) : 0.0;
  } else if (q < L.theta()) {
    const int e = q - L.c0(), f = e / NG, i = e % NG;
    // fields c0, s0, i0r, i0i, res, dmp, inv2h in canonical order
    const int64_t base[7] = {C.c0(), C.s0(), C.i0r(), C.i0i(), C.res(), C.dmp(), C.inv2h()};
    if (i < n) {
      v = cn[base[f] + i];
      if (rotated && (f == 2 || f == 3)) {
        const double2 J = cmul(conj_emf(i), make_double2(cn[C.i0r() + i], cn[C.i0i() + i]));
        v = f == 2 ? J.x : J.y;
      }
      if (f >= 2 && f <= 5) v *= scale(i);
    }
  } else if (q >= L.owner()) {
    const int p = q - L.owner();
    v = p < P ? (double)owner[p] : -1.0;
  } else {
    const int e = q - L.theta(), f = e / PM, p = e % PM;
    const int64_t base[3] = {C.theta(), C.sigma(), C.xi0()};
    if (p < P) v = cn[base[f] + p];
  }
  coef[q] = (R)v;
}

template <typename R>
hipError_t launch_pack(const double* canon, int n, int P, const int32_t* gen,
                       const int32_t* owner, bool rotated, int NG, int PM, R* coef, hipStream_t st) {
  PackLayout L{NG, PM};
  hipLaunchKernelGGL(k_pack<R>, dim3((L.size() + 255) / 256), dim3(256), 0, st, canon, n, P, gen,
                     owner, rotated, NG, PM, coef);
  return hipGetLastError();
}
template hipError_t launch_pack<double>(const double*, int, int, const int32_t*, const int32_t*,
                                        bool, int, int, double*, hipStream_t);
template hipError_t launch_pack<float>(const double*, int, int, const int32_t*, const int32_t*, bool,
                                       int, int, float*, hipStream_t);

// Ordered merge of per-group statistics into mean and variance (Alg. 1 step
// 4): partial[g * gstride + q] holds (mean, M2) of group g's samples for
// q = row * V + v (group_size samples per group, the last group the rest).
// A workgroup takes 64 consecutive q, one per lane, and splits the groups
// into kMergeSplit contiguous ranges, one per wave: each wave merges its
// range in group order with Chan's update (loads eight groups ahead, so
// that about 10 MB of partials are in flight over the workgroups), then
// the first wave merges the waves' results in wave order.  The order depends
// only on the sizes, so repeated runs give the same bits; every wave reads
// 64 consecutive pairs (1 KB) per group, and the workgroups together stream
// the partials once.  Angles get delta0 back (the integrators work in
// deviations).
constexpr int kMergeSplit = 16;

__device__ __forceinline__ void chan_merge(double& cnt, double& m, double& M2, double nb,
                                           double mb, double M2b) {
  const double tot = cnt + nb;
  const double dlt = mb - m;
  const double fb = tot > 0.0 ? nb / tot : 0.0;
  m += dlt * fb;
  M2 += M2b + dlt * dlt * (cnt * fb);
  cnt = tot;
}

__global__ void __launch_bounds__(64 * kMergeSplit) k_stats_merge(
    const double2* __restrict__ partial, int64_t gstride, int64_t n_groups, int group_size,
    int64_t N, int64_t SV, int V, int n, int ddof, const double* __restrict__ delta0,
    double* __restrict__ mean, double* __restrict__ var) {
  __shared__ double sh[3][kMergeSplit][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t q = (int64_t)blockIdx.x * 64 + lane;
  const bool on = q < SV;
  const int64_t per = (n_groups + kMergeSplit - 1) / kMergeSplit;
  const int64_t g0 = wv * per, g1 = g0 + per < n_groups ? g0 + per : n_groups;
  double cnt = 0.0, m = 0.0, M2 = 0.0;
  const double2* src = partial + (on ? q : 0);
  constexpr int D = 8;
  for (int64_t g = g0; g < g1; g += D) {
    double2 pt[D];
#pragma unroll
    for (int u = 0; u < D; ++u) pt[u] = (on && g + u < g1) ? src[(g + u) * gstride] : double2{0.0, 0.0};
#pragma unroll
    for (int u = 0; u < D; ++u) {
      if (g + u >= g1) break;
      const int64_t rem = N - (g + u) * group_size;
      chan_merge(cnt, m, M2, (double)(rem < group_size ? rem : group_size), pt[u].x, pt[u].y);
    }
  }
  sh[0][wv][lane] = cnt;
  sh[1][wv][lane] = m;
  sh[2][wv][lane] = M2;
  __syncthreads();
  if (wv != 0 || !on) return;
  for (int w = 1; w < kMergeSplit; ++w)
    chan_merge(cnt, m, M2, sh[0][w][lane], sh[1][w][lane], sh[2][w][lane]);
  const int v = (int)(q % V);
  mean[q] = m + (v < n ? delta0[v] : 0.0);
  var[q] = M2 / (double)(N - ddof);
}

hipError_t launch_stats_merge_rows(const double2* partial, int64_t gstride, int64_t n_groups,
                                   int group_size, int64_t N, int64_t rows, int V, int n,
                                   int ddof, const double* delta0, double* mean, double* var,
                                   hipStream_t st) {
  const int64_t SV = rows * V;
  if (SV <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_stats_merge, dim3((unsigned)((SV + 63) / 64)), dim3(64 * kMergeSplit), 0,
                     st, partial, gstride, n_groups, group_size, N, SV, V, n, ddof, delta0, mean,
                     var);
  return hipGetLastError();
}

hipError_t launch_stats_merge(const double2* partial, int64_t n_groups, int group_size,
                              int64_t N, int64_t S, int V, int n, int ddof,
                              const double* delta0, double* mean, double* var, hipStream_t st) {
  return launch_stats_merge_rows(partial, (S + 1) * V, n_groups, group_size, N, S + 1, V, n, ddof,
                                 delta0, mean, var, st);
}

}  // namespace fmc
