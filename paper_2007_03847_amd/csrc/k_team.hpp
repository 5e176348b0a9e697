// k_team.hpp -- classical machines, one tile of 16 trajectories per workgroup,
// the network product on the matrix cores: fmc_run above ten machines, and the
// matrix-core variants of the batched and served forms (FP32).
//
// Same deviation form as the other integrators of classical machines: in FP64 the
// rotated form of the coefficients (PackLayout), eps = e^{j d} - 1 and the network
// part sum_k Z_ik eps_k; in FP32 the plain one, Y for Z and E0 eps for eps
// (rotated_form).  The workgroup is a team of NB waves; wave v owns the eight
// machines 8 v .. 8 v + 7 of the tile's 16 trajectories.  Their sums are one
// 16 x 16 block of a real product W x, where the vector x interleaves
// (1 - cos d, sin d) machine by machine and W is made of the 2 x 2 blocks
// [-Zr -Zi; -Zi Zr], on
// v_mfma_f64_16x16x4 or v_mfma_f32_16x16x4.  The rows of a block are ordered so
// that the accumulator leaves lane l with Re and Im of the machines 8 v + 2 (l/16)
// and the next one of trajectory l%16: the lane that receives the sums holds
// those machines' states.  A wave's 16 rows of W stay in registers (2 NG values in
// 2 NG / 4 fragments), x goes through LDS.
//
// Two exchanges per step: an angle's derivative is its speed, so the angles of
// stages 1 and 2 are known at the start of a step and those of stages 3 and 4
// once the accelerations of 1 and 2 are.  Each pair of stages shares one rotation,
// one barrier and one pass over the fragments of W, as two independent chains of
// matrix operations.
//
// Why this split.  The lanes-per-trajectory kernel keeps a row of Y per lane and
// spills from 24 machines on in FP64 (37 machines, 3001 samples, 1000 steps:
// 197 ms per call, 200 registers of spill traffic in every stage); here the
// product is the matrix pipe's and a lane holds two machines.  A block of eight
// machines pads n to a multiple of 8, where separate real and imaginary blocks
// of 16 would pad to 16 (37 machines: 100 against 144 matrix operations per
// tile and stage).  The team splits a tile's machines over waves so that a few
// thousand samples fill the chip: 3001 samples are 188 tiles, 940 waves for 1024
// SIMDs.  Bound by the FP64 matrix pipe (64 cycles per operation) when several
// teams share a SIMD, by the chain of a pair (rotation, barrier, 2 NG / 4
// dependent matrix operations on each of two chains) when one does.
#pragma once

#include <hip/hip_runtime.h>

#include "fmc_internal.hpp"
#include "k_integrate.hpp"

namespace fmc {

constexpr int kTeamT = 16;  // trajectories per tile
constexpr int kTeamPM = 8;  // process slots

typedef double d4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

template <typename R> struct TeamMma;
template <> struct TeamMma<double> {
  using acc = d4v;
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // result register r of lane l is row 4 r + l/16: the (machine pair, register) of row i
  static __device__ __forceinline__ int pair(int i) { return i & 3; }
  static __device__ __forceinline__ int reg(int i) { return i >> 2; }
};
template <> struct TeamMma<float> {
  using acc = f4v;
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // row 4 (l/16) + r
  static __device__ __forceinline__ int pair(int i) { return i >> 2; }
  static __device__ __forceinline__ int reg(int i) { return i & 3; }
};

// Output steps collected before they are reduced: a row each for most of the
// team's threads; more steps take LDS from the teams that share a CU.
constexpr int kTeamSteps = 2;
// Values of a tile's state between chunks.
__host__ __device__ constexpr int team_state(int NB) { return 4 * 64 * NB + (kTeamPM + 2) * kTeamT; }

// Exchange buffers: two in turn need one barrier per pair of stages; the larger
// teams take one (and a second barrier) to keep two teams on a CU.
template <int NB, int TW>
constexpr int team_buffers() {
  return NB <= 4 && TW == 1 ? 2 : 1;
}

// LDS of a workgroup of TW teams.
template <typename R, int NB, int TW>
struct TeamLds {
  static constexpr int VM = 16 * NB + kTeamPM, XB = team_buffers<NB, TW>(), T = kTeamT * TW;
  // x of each team's tile in two stages: row 2 m of machine m holds 1 - cos d, row
  // 2 m + 1 sin d; and the processes' stage values (row kTeamPM stays zero)
  R X[TW][XB][2][16 * NB][kTeamT];
  R XI[TW][XB][2][kTeamPM + 1][kTeamT];
  double tile[kTeamSteps][VM][T + 1];
  R s_ref[TW][NB][kTeamT];  // each wave's sum of the angles of its machines
  int s_bad[T];
};

// TW teams of NB waves: trajectories 16 TW tl .. 16 TW (tl + 1) - 1 over the steps
// [s_begin, s_end) of a, machines packed for NG; st as in group_run.
template <typename R, int NB, int TW>
__device__ __forceinline__ void team_run(const IntegArgs<R>& a, int NG, int64_t tl,
                                         TeamLds<R, NB, TW>& S, GroupStats st) {
  using M = TeamMma<R>;
  constexpr int PM = kTeamPM, KS = 4 * NB, D = kTeamSteps;
  constexpr int XB = team_buffers<NB, TW>(), T = kTeamT * TW, TPB = 64 * NB * TW;
  const PackLayout Lp{NG, PM};
  // opaque, so that a persistent kernel's tile loop does not keep every address of
  // the set-up below in registers
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), team = wave / NB, wv = wave - team * NB;
  const int l = tid & 63, g = l >> 4, t = l & 15;
  auto& X = S.X[team];
  auto& XI = S.XI[team];
  auto& tile = S.tile;
  auto& s_ref = S.s_ref[team];
  auto& s_bad = S.s_bad;
  const int n = a.n, P = a.P, V = a.V;
  const int64_t N = a.N;
  const int tt = team * kTeamT + t;  // my trajectory of the workgroup's
  const int64_t traj = tl * T + tt;
  const bool valid = traj < N;
  const int64_t ns = valid ? traj : N - 1;
  const int64_t rem = N - tl * T;
  const int cnt = rem < T ? (int)rem : T;
  const R* __restrict__ cf = a.coef;
  const R* __restrict__ w = a.w;
  const int slot = (valid && a.traj_slot) ? a.traj_slot[ns] : -1;

  // the wave's rows of W as A fragments: lane l holds row l%16, column 4 s + l/16
  R yv[KS];
  {
    const int mi = 8 * wv + 2 * M::pair(t) + (M::reg(t) >> 1), ci = M::reg(t) & 1;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int mk = 2 * s + (g >> 1), ck = g & 1;
      const bool on = mi < NG && mk < NG;
      const int64_t e = on ? (int64_t)mi * NG + mk : 0;
      const R zr = on ? cf[Lp.yre() + e] : R(0), zi = on ? cf[Lp.yim() + e] : R(0);
      yv[s] = ci != ck ? -zi : (ci == 0 ? -zr : zr);
    }
  }
  // my two machines
  constexpr bool ROT = rotated_form<R>();
  R jr[2], ji[2], res[2], dmp[2], e0r[2], e0i[2], inv2h[2];
  bool live[2], on[2];
  int live_mask[2];
  int pq[2];         // the first process at the machine, PM if none
  R bin[2];          // the machine's injection factor
  bool more = false;  // a machine of this wave has several processes
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int m = 8 * wv + 2 * g + q;
    const bool in = m < NG;
    jr[q] = in ? cf[Lp.i0r() + m] : R(0);
    ji[q] = in ? cf[Lp.i0i() + m] : R(0);
    res[q] = in ? cf[Lp.res() + m] : R(0);
    dmp[q] = in ? cf[Lp.dmp() + m] : R(0);
    e0r[q] = ROT ? R(1) : (in ? cf[Lp.c0() + m] : R(0));
    e0i[q] = ROT ? R(0) : (in ? cf[Lp.s0() + m] : R(0));
    inv2h[q] = ROT ? R(1) : (in ? cf[Lp.inv2h() + m] : R(0));
    on[q] = m < n;
    live[q] = in && (cf[Lp.c0() + m] != R(0) || cf[Lp.s0() + m] != R(0));  // in service
    live_mask[q] = lane_mask(live[q]);
    pq[q] = PM;
    bin[q] = R(0);
    for (int p = PM - 1; p >= 0; --p)
      if (in && cf[Lp.binc() + m * PM + p] != R(0)) {
        more = more || pq[q] != PM;
        pq[q] = p;
        bin[q] = cf[Lp.binc() + m * PM + p];
      }
  }
  more = __builtin_amdgcn_ballot_w64(more) != 0;
  // my process: 4 wv + g of trajectory t
  const int pr = 4 * wv + g;
  const bool own = pr < P;
  const int own_mask = lane_mask(own);
  const R theta = own ? cf[Lp.theta() + pr] : R(0), sigma = own ? cf[Lp.sigma() + pr] : R(0);
  const int64_t wofs = own ? (int64_t)pr * N + ns : 0, colstride = (int64_t)P * N;
  for (int q = tid; q < TW * XB * 2 * (PM + 1) * kTeamT; q += TPB) (&S.XI[0][0][0][0][0])[q] = R(0);
  __syncthreads();

  R yd[2], yw[2], yx;
  double coff = 0.0;  // common-angle offset of the trajectory (see IntegArgs::recenter)
  // State between chunks (team_state values per tile): angles and speeds [4][64 NB],
  // the processes [8][16], the offset's two slots [2][16]
  const int64_t sb = (tl * TW + team) * team_state(NB), sp = sb + 4 * 64 * NB, so = sp + PM * kTeamT + t;
  if (a.s_begin == 0) {
    yd[0] = yd[1] = yw[0] = yw[1] = R(0);
    yx = own ? cf[Lp.xi0() + pr] : R(0);
  } else {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      yd[q] = a.state[sb + q * 64 * NB + 64 * wv + l];
      yw[q] = a.state[sb + (2 + q) * 64 * NB + 64 * wv + l];
    }
    yx = own ? a.state[sp + pr * kTeamT + t] : R(0);
    coff = load_offset(a.state, so, so + kTeamT);
  }
  double racc = 0.0;  // RRF sum of trajectory tid (threads tid < cnt; see IntegArgs::rrf_w)
  if (a.rrf_w && a.s_begin > 0 && tid < cnt) racc = a.rrf_acc[tl * T + tid];

  int nbuf = 0;
  int64_t s_first = 0;
  auto flush = [&]() {
    __syncthreads();
    // TW neighbouring lanes per row (step, variable), 16 samples each
    const int h = tid % TW;
    const int mine = cnt - kTeamT * h < kTeamT ? cnt - kTeamT * h : kTeamT;
    for (int rv = tid / TW; rv < nbuf * V; rv += TPB / TW) {
      const int b = rv / V, v = rv - b * V;
      double mu = 0.0, m2 = 0.0;
      if (mine > 0) row_stats(&tile[b][v][kTeamT * h], mine, mu, m2);
#pragma unroll
      for (int e = 1; e < TW; e *= 2) {  // Chan's update, pairs then pairs of pairs
        const double muo = __shfl_xor(mu, e, 64), m2o = __shfl_xor(m2, e, 64);
        const int c0 = cnt - kTeamT * (h & ~(2 * e - 1)), ca = c0 < kTeamT * e ? c0 : kTeamT * e;
        const int cb = c0 - ca < kTeamT * e ? c0 - ca : kTeamT * e;
        if ((h & e) == 0 && cb > 0) {
          const double dl = muo - mu, tot = (double)(ca + cb);
          mu += dl * ((double)cb / tot);
          m2 += m2o + dl * dl * ((double)ca * (double)cb / tot);
        }
      }
      if (h != 0) continue;
      double2* dst = st.rows + (s_first + b) * V + v;
      if (st.prev == 0) {
        *dst = make_double2(mu, m2);
      } else {
        const double2 old = *dst;
        const double na = (double)st.prev, nb = (double)cnt, tot = na + nb, dl = mu - old.x;
        *dst = make_double2(old.x + dl * (nb / tot), old.y + m2 + dl * dl * (na * nb / tot));
      }
    }
    if (a.rrf_w && tid < cnt) {
      for (int b = 0; b < nbuf; ++b) {
        const int64_t s = s_first + b;
        double u = 0.0;
        for (int v = 0; v < V; ++v) {
          const double y = tile[b][v][tid];
          u += a.rrf_w[v] * (v < n ? a.delta0[v] + y : y);
        }
        racc += (s == 0 || s == a.S ? 0.5 : 1.0) * u * u;
      }
    }
    __syncthreads();
    nbuf = 0;
  };
  // Where my outputs go in a collected step's rows: machines and processes that
  // do not exist write the padding column, so that no lane branches.
  constexpr int RS = T + 1;
  int od[2], ow[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int m = 8 * wv + 2 * g + q;
    od[q] = on[q] ? m * RS + tt : T;
    ow[q] = on[q] ? (n + m) * RS + tt : T;
  }
  const int ox = own ? (2 * n + pr) * RS + tt : T;
  const bool traced = __builtin_amdgcn_ballot_w64(slot >= 0) != 0;  // some lane stores a trajectory
  auto emit = [&](int64_t s) {
    if (nbuf == 0) s_first = s;
    double* tb = &tile[nbuf][0][0];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      tb[od[q]] = coff + (double)yd[q];
      tb[ow[q]] = (double)yw[q];
    }
    tb[ox] = (double)yx;
    if (traced && slot >= 0) {
      double* o = a.traj + ((int64_t)slot * (a.S + 1) + s) * V;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int m = 8 * wv + 2 * g + q;
        if (on[q]) {
          o[m] = a.delta0[m] + (coff + (double)yd[q]);
          o[n + m] = (double)yw[q];
        }
      }
      if (own) o[2 * n + pr] = (double)yx;
    }
    if (++nbuf == D) flush();  // nbuf is uniform over the workgroup
  };
  if (a.s_begin == 0) emit(0);

  int buf = 0;
  // Network part of a pair of stages at angles d[h] and process values x[h]: the
  // sums of my machines (registers 2 q, 2 q + 1 of cur[h])
  R sd[2][2], omc[2][2];
  typename M::acc cur[2];
  auto network = [&](const R (&d)[2][2], R x0, R x1) {
    if constexpr (XB == 1)
      __syncthreads();  // every wave has read the previous pair
    else
      buf ^= 1;
    rotation_stages<R, 2, 2>(d, live, live_mask, sd, omc);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (!ROT) {
#pragma unroll
        for (int q = 0; q < 2; ++q) turn(e0r[q], e0i[q], omc[h][q], sd[h][q]);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        // a machine without EMF has a zero column of Z and turns by zero
        X[buf][h][16 * wv + 4 * g + 2 * q][t] = omc[h][q];
        X[buf][h][16 * wv + 4 * g + 2 * q + 1][t] = sd[h][q];
      }
    }
    if (own) {
      XI[buf][0][pr][t] = x0;
      XI[buf][1][pr][t] = x1;
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) cur[h] = typename M::acc{R(0), R(0), R(0), R(0)};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int h = 0; h < 2; ++h) cur[h] = M::mma(yv[s], X[buf][h][4 * s + g][t], cur[h]);
    }
  };
  // accelerations of my machines in stage h at speeds u
  auto accel = [&](int h, const R (&u)[2], R (&acc)[2]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      R inj = XI[buf][h][pq[q]][t];
      if (more) {  // wave-uniform: add every further process of my machines
        const int m = 8 * wv + 2 * g + q;
#pragma unroll 1
        for (int p = pq[q] + 1; p < PM; ++p)
          if (m < NG && cf[Lp.binc() + m * PM + p] != R(0)) inj += XI[buf][h][p][t];
      }
      R F = res[q] - dmp[q] * u[q] + bin[q] * inj;
      F = fma(omc[h][q], jr[q], F);
      F = fma(-sd[h][q], ji[q], F);
      if constexpr (ROT) {
        F = fma(omc[h][q] - R(1), cur[h][2 * q], F);
        acc[q] = fma(-sd[h][q], cur[h][2 * q + 1], F);
      } else {
        F = fma(omc[h][q] - e0r[q], cur[h][2 * q], F);
        F = fma(-(e0i[q] + sd[h][q]), cur[h][2 * q + 1], F);
        acc[q] = F * inv2h[q];
      }
    }
  };

  const R dt = a.dt, h2 = a.dt * R(0.5), dt6 = a.dt / R(6);
  const R hw2 = h2 * a.wb, hw = dt * a.wb;
  const R inv_n = R(1) / (R)a.n_ref;
  // the next step's path values load a step ahead; a lane without a process loads
  // the first one's of the first sample and masks it (its sigma is zero, that path
  // may not be finite), the last step its own columns again
  R w0 = w[wofs], w1 = w[colstride + wofs], w2 = w[2 * colstride + wofs];
  w0 = masked(own_mask, w0);
  for (int64_t s = a.s_begin; s < a.s_end; ++s) {
    w1 = masked(own_mask, w1);
    w2 = masked(own_mask, w2);
    const int64_t cn = 2 * (s + 1 < a.s_end ? s + 1 : s) - a.c_base;  // first column of the next step
    const R n1 = w[(cn + 1) * colstride + wofs], n2 = w[(cn + 2) * colstride + wofs];
    // the four stage values of my process (it does not see the machines)
    const R k1 = sigma * w0 - theta * yx;
    const R x2 = yx + h2 * k1, k2 = sigma * w1 - theta * x2;
    const R x3 = yx + h2 * k2, k3 = sigma * w1 - theta * x3;
    const R x4 = yx + dt * k3, k4 = sigma * w2 - theta * x4;
    // the angles' derivatives are w_b times the stage speeds
    R d[2][2], u[2], v[2], k[2], sa[2], su[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      d[0][q] = yd[q];
      d[1][q] = yd[q] + hw2 * yw[q];
    }
    network(d, yx, x2);
    accel(0, yw, k);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      u[q] = yw[q] + h2 * k[q];
      su[q] = yw[q] + R(2) * u[q];
      sa[q] = k[q];
      d[0][q] = yd[q] + hw2 * u[q];
    }
    accel(1, u, k);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      v[q] = yw[q] + h2 * k[q];
      su[q] += R(2) * v[q];
      sa[q] += R(2) * k[q];
      d[1][q] = yd[q] + hw * v[q];
    }
    network(d, x3, x4);
    accel(0, v, k);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      u[q] = yw[q] + dt * k[q];
      su[q] += u[q];
      sa[q] += R(2) * k[q];
    }
    accel(1, u, k);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      yd[q] += angle_step(dt6, a.wb, su[q]);
      yw[q] += dt6 * (sa[q] + k[q]);
    }
    yx += dt6 * (((k1 + R(2) * k2) + R(2) * k3) + k4);
    w0 = w2;
    w1 = n1;
    w2 = n2;
    if (a.recenter && ((s + 1) & 7) == 0) {
      // every eighth step of the absolute count (time chunks keep the bits): the
      // mean angle of the machines in service goes into the offset.  Lanes t,
      // t + 16, t + 32, t + 48 hold the wave's machines of trajectory t; the waves'
      // sums are added in wave order by every lane.
      R part = (live[0] ? yd[0] : R(0)) + (live[1] ? yd[1] : R(0));
      R sum = __shfl(part, t, 64);
      sum += __shfl(part, t + 16, 64);
      sum += __shfl(part, t + 32, 64);
      sum += __shfl(part, t + 48, 64);
      if (g == 0) s_ref[wv][t] = sum;
      __syncthreads();
      sum = s_ref[0][t];
#pragma unroll
      for (int v = 1; v < NB; ++v) sum += s_ref[v][t];
      const R ref = sum * inv_n;
      coff += (double)ref;
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (on[q]) yd[q] -= ref;
    }
    emit(s + 1);
  }
  if (nbuf > 0) flush();
  if (a.rrf_w && tid < cnt) {
    a.rrf_acc[tl * T + tid] = racc;
    if (a.s_end == a.S) a.rrf[tl * T + tid] = sqrt(racc / (double)a.S);
  }
  if (a.state) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      a.state[sb + q * 64 * NB + 64 * wv + l] = yd[q];
      a.state[sb + (2 + q) * 64 * NB + 64 * wv + l] = yw[q];
    }
    if (own) a.state[sp + pr * kTeamT + t] = yx;
    if (wv == 0 && g == 0) store_offset(a.state, so, so + kTeamT, coff);
  }

  if (a.s_end == a.S) {  // uniform: one count per trajectory with a non-finite state
    bool bad = !isfinite(coff) || !isfinite(yx);
#pragma unroll
    for (int q = 0; q < 2; ++q) bad |= !isfinite(yd[q]) || !isfinite(yw[q]);
    if (tid < T) s_bad[tid] = 0;
    __syncthreads();
    if (bad) s_bad[tt] = 1;
    __syncthreads();
    if (tid < cnt && s_bad[tid] != 0) {
      atomicAdd(a.nonfinite, 1ULL);
      atomicMin(a.first_bad, (long long)(tl * T + tid));
    }
  }
  __syncthreads();  // the LDS is free for the workgroup's next tile
}

}  // namespace fmc
