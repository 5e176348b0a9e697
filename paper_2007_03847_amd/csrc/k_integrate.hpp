// k_integrate.hpp -- batched fixed-step integrator of the classical
// multimachine model driven by the KLE-rebuilt OU disturbances (eq. 9 in the
// swing equations, Alg. 1 steps 2-3), with the cross-sample statistics of
// Alg. 1 step 4 fused into its epilogue.
//
// One trajectory per lane.  The machine data (reduced admittance, operating
// point) is identical for every lane of a wave, so it is read through uniform
// (scalar) loads and feeds the FMAs as scalar operands: no LDS or VGPR traffic
// for Y.
//
// The state is integrated as deviations from the operating point:
//   y = (d_delta_i, dw_i, xi_p).
// With E~_k = E~0_k exp(j d_delta_k), exp(j d) - 1 = -2 sin^2(d/2) + j sin d,
// so dE~ = E~0 (exp(j d) - 1) is formed from one sincos of d/2 without
// cancellation, and
//   Pe_i - Pe0_i = Re(dE~_i conj(I0_i)) + Re(E~_i conj(dI_i)),  dI = Y dE~,
// which keeps FP32 integration accurate to its own rounding of the deviation.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "fmc_internal.hpp"

namespace fmc {

// Read-only machine data seen through the constant address space: uniform
// loads from it become scalar (SMEM) loads into SGPRs.
template <typename R>
using cptr = const __attribute__((address_space(4))) R*;

// sin and cos together (sincos_r_nb): Cody-Waite reduction x = k pi/2 + r,
// |r| <= pi/4, with pi/2 split into two (FP64) or three (FP32) parts applied
// by FMA (exact enough for |k| < 2^20, far beyond the angles met here), then
// the Taylor polynomials of sin and cos in r^2 (terms through r^15 / r^16 in
// FP64, r^9 / r^10 in FP32; truncation below half an ulp on |r| <= pi/4), and
// the quadrant of k.
__device__ __forceinline__ bool sincos_all_small(bool small) {
  return __builtin_amdgcn_ballot_w64(!small) == 0;
}

// a*b + c as the three-operand FMA with the coefficient c in a scalar register
// pair: the coefficients take no vector registers and no copies (the
// two-operand form ties the addend to the result and costs a copy of the
// coefficient per use)
__device__ __forceinline__ double fma3(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

// the polynomials on the reduced argument r
__device__ __forceinline__ void sincos_poly(double r, double& sr, double& cr) {
  auto f = [](double a, double b, double c) { return fma(a, b, c); };
  const double r2 = r * r;
  double ps = -1.0 / 1307674368000.0;
  ps = f(ps, r2, 1.0 / 6227020800.0);
  ps = f(ps, r2, -1.0 / 39916800.0);
  ps = f(ps, r2, 1.0 / 362880.0);
  ps = f(ps, r2, -1.0 / 5040.0);
  ps = f(ps, r2, 1.0 / 120.0);
  ps = f(ps, r2, -1.0 / 6.0);
  sr = fma(r * r2, ps, r);
  double pc = 1.0 / 20922789888000.0;
  pc = f(pc, r2, -1.0 / 87178291200.0);
  pc = f(pc, r2, 1.0 / 479001600.0);
  pc = f(pc, r2, -1.0 / 3628800.0);
  pc = f(pc, r2, 1.0 / 40320.0);
  pc = f(pc, r2, -1.0 / 720.0);
  pc = f(pc, r2, 1.0 / 24.0);
  pc = fma(pc, r2, -0.5);
  cr = fma(r2, pc, 1.0);
}

__device__ __forceinline__ void sincos_poly(float r, float& sr, float& cr) {
  const float r2 = r * r;
  float ps = 1.0f / 362880.0f;
  ps = fmaf(ps, r2, -1.0f / 5040.0f);
  ps = fmaf(ps, r2, 1.0f / 120.0f);
  ps = fmaf(ps, r2, -1.0f / 6.0f);
  sr = fmaf(r * r2, ps, r);
  float pc = -1.0f / 3628800.0f;
  pc = fmaf(pc, r2, 1.0f / 40320.0f);
  pc = fmaf(pc, r2, -1.0f / 720.0f);
  pc = fmaf(pc, r2, 1.0f / 24.0f);
  pc = fmaf(pc, r2, -0.5f);
  cr = fmaf(r2, pc, 1.0f);
}

// The reduction always taken, with no branch: for callers that evaluate the
// sin/cos of several machines per lane back to back, where a branch per call
// would keep the compiler from interleaving them.
__device__ __forceinline__ void sincos_r_nb(double x, double& s, double& c) {
  const double k = rint(x * 0.63661977236758134308);  // 2/pi
  double r = fma(-k, 0x1.921fb54442d18p+0, x);
  r = fma(-k, 0x1.1a62633145c07p-54, r);
  double sr, cr;
  sincos_poly(r, sr, cr);
  const int q = (int)k;
  const double a = (q & 1) ? cr : sr;
  const double b = (q & 1) ? sr : cr;
  s = (q & 2) ? -a : a;
  c = ((q + 1) & 2) ? -b : b;
}

__device__ __forceinline__ void sincos_r_nb(float x, float& s, float& c) {
  const float k = rintf(x * 0x1.45f306p-1f);  // 2/pi
  float r = fmaf(-k, 0x1.921fb6p+0f, x);
  r = fmaf(-k, -0x1.777a5cp-25f, r);
  r = fmaf(-k, -0x1.ee59dap-50f, r);
  float sr, cr;
  sincos_poly(r, sr, cr);
  const int q = (int)k;
  const float a = (q & 1) ? cr : sr;
  const float b = (q & 1) ? sr : cr;
  s = (q & 2) ? -a : a;
  c = ((q + 1) & 2) ? -b : b;
}

// sin d and 1 - cos d of a lane's angle deviations d (of N machines in M stages).  When every active
// lane's angles are below half a radian (the usual case for deviations from the
// operating point), both come straight from their Taylor polynomials in d^2
// (sin through d^13 and 1 - cos through d^14 in FP64, d^7 and d^8 in FP32: the
// first term left out is below half an ulp), 15 operations in FP64 against 23
// for the half-angle form below, and without its doubled rounding; else from
// one sin/cos of d/2 with the full reduction, 1 - cos d = 2 sin^2(d/2), which
// has no cancellation either.  live[k] = false marks a machine without EMF (or an
// idle lane): its angle does not decide the branch, and it turns by zero (see
// masked), since whatever its angle has become multiplies a zero.
__device__ __forceinline__ void rotation_poly(double d, double& sd, double& omc) {
  const double r2 = d * d;
  double ps = 1.0 / 6227020800.0;
  ps = fma3(ps, r2, -1.0 / 39916800.0);
  ps = fma3(ps, r2, 1.0 / 362880.0);
  ps = fma3(ps, r2, -1.0 / 5040.0);
  ps = fma3(ps, r2, 1.0 / 120.0);
  ps = fma3(ps, r2, -1.0 / 6.0);
  sd = fma(d * r2, ps, d);
  double pc = 1.0 / 87178291200.0;
  pc = fma3(pc, r2, -1.0 / 479001600.0);
  pc = fma3(pc, r2, 1.0 / 3628800.0);
  pc = fma3(pc, r2, -1.0 / 40320.0);
  pc = fma3(pc, r2, 1.0 / 720.0);
  pc = fma3(pc, r2, -1.0 / 24.0);
  pc = fma(pc, r2, 0.5);
  omc = r2 * pc;
}
__device__ __forceinline__ void rotation_poly(float d, float& sd, float& omc) {
  const float r2 = d * d;
  float ps = -1.0f / 5040.0f;
  ps = fmaf(ps, r2, 1.0f / 120.0f);
  ps = fmaf(ps, r2, -1.0f / 6.0f);
  sd = fmaf(d * r2, ps, d);
  float pc = -1.0f / 40320.0f;
  pc = fmaf(pc, r2, 1.0f / 720.0f);
  pc = fmaf(pc, r2, -1.0f / 24.0f);
  pc = fmaf(pc, r2, 0.5f);
  omc = r2 * pc;
}
// v where the mask is set, else zero: in FP64 a number below 2^-1042, since the high
// word alone is masked.  For values that a zero multiplies later, which would not
// remove an infinity or a NaN.  The group and team integrators keep the mask in a
// vector register (lane_mask): as a condition it would be one of the scalar register
// pairs that they spill already, and a pair comes back by way of two lane reads
// (10 machines, 1e4 samples, 4000 FP64 steps: 9.37 ms, 9.16 here, 9.05 unmasked).
__device__ __forceinline__ int lane_mask(bool on) {
  int m = on ? -1 : 0;
  asm("" : "+v"(m));
  return m;
}
__device__ __forceinline__ float masked(int mask, float v) {
  return __int_as_float(__float_as_int(v) & mask);
}
__device__ __forceinline__ double masked(int mask, double v) {
  return __hiloint2double(__double2hiint(v) & mask, __double2loint(v));
}
__device__ __forceinline__ float masked(bool on, float v) { return on ? v : 0.0f; }
__device__ __forceinline__ double masked(bool on, double v) {
  return __hiloint2double(on ? __double2hiint(v) : 0, __double2loint(v));
}
template <typename R, int M, int N, typename Mask>
__device__ __forceinline__ void rotation_stages(const R (&d)[M][N], const bool (&live)[N],
                                                const Mask (&mask)[N], R (&sd)[M][N], R (&omc)[M][N]) {
  bool small = true;
#pragma unroll
  for (int h = 0; h < M; ++h)
#pragma unroll
    for (int k = 0; k < N; ++k) small = small && (!live[k] || fabs(d[h][k]) < R(0.5));
  if (sincos_all_small(small)) [[likely]] {
#pragma unroll
    for (int h = 0; h < M; ++h)
#pragma unroll
      for (int k = 0; k < N; ++k) rotation_poly(masked(mask[k], d[h][k]), sd[h][k], omc[h][k]);
  } else {
#pragma unroll
    for (int h = 0; h < M; ++h)
#pragma unroll
      for (int k = 0; k < N; ++k) {
        R sh, ch;
        sincos_r_nb(live[k] ? d[h][k] * R(0.5) : R(0), sh, ch);
        sd[h][k] = R(2) * sh * ch;
        omc[h][k] = R(2) * sh * sh;
      }
  }
}
template <typename R, int N>
__device__ __forceinline__ void rotation_many(const R (&d)[N], const bool (&live)[N], R (&sd)[N],
                                              R (&omc)[N]) {
  using A = const R (*)[1][N];
  using B = R (*)[1][N];
  rotation_stages<R, 1, N>(*(A)&d, live, live, *(B)&sd, *(B)&omc);
}

// The FP64 common-angle offset in two state slots: the exact bits of the
// double (two 32-bit halves for an FP32 state array), so that a run split
// into time chunks gives the same bits as a run in one chunk.
__device__ __forceinline__ void store_offset(float* st, int64_t i0, int64_t i1, double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  reinterpret_cast<unsigned int*>(st)[i0] = (unsigned int)b;
  reinterpret_cast<unsigned int*>(st)[i1] = (unsigned int)(b >> 32);
}
__device__ __forceinline__ void store_offset(double* st, int64_t i0, int64_t, double v) {
  st[i0] = v;
}
__device__ __forceinline__ double load_offset(const float* st, int64_t i0, int64_t i1) {
  const unsigned long long lo = reinterpret_cast<const unsigned int*>(st)[i0];
  const unsigned long long hi = reinterpret_cast<const unsigned int*>(st)[i1];
  return __longlong_as_double((long long)(lo | (hi << 32)));
}
__device__ __forceinline__ double load_offset(const double* st, int64_t i0, int64_t) {
  return st[i0];
}

// d xi/dt of eq. 9 for a general Ito process whose row q sits in registers; root
// and poly (wave-uniform): some lane has a process with a square-root or a
// polynomial diffusion, so that a wave pays only for the forms it has.
template <typename R>
__device__ __forceinline__ R sde_rate(const R (&q)[kSdeCols], R x, R w, bool root, bool poly) {
  const R mu = q[SDE_M0] + x * (q[SDE_M1] + x * q[SDE_M2]);
  R sg = R(0), ssp = R(0);  // sigma and sigma sigma'
  if (poly) {
    sg = q[SDE_C0] + x * (q[SDE_C1] + x * q[SDE_C2]);
    ssp = sg * (q[SDE_C1] + R(2) * q[SDE_C2] * x);
  }
  if (root) {
    const R d = x - q[SDE_R];
    const R g = q[SDE_C0] + x * (q[SDE_C1] + x * q[SDE_C2]) + q[SDE_C3] * fabs(d);
    const R sgn = d > R(0) ? R(1) : (d < R(0) ? R(-1) : R(0));
    const R dg = q[SDE_C1] + R(2) * q[SDE_C2] * x + q[SDE_C3] * sgn;
    const bool pos = g > R(0), mine = q[SDE_FORM] == R(2);
    sg = mine ? (pos ? sqrt(g) : R(0)) : sg;
    ssp = mine ? (pos ? R(0.5) * dg : R(0)) : ssp;
  }
  return mu - q[SDE_K] * ssp + sg * w;
}

// d xi/dt of eq. 9 for a general Ito process (one row of IntegArgs::sde) at
// state x with white-noise surrogate value w, and the power it injects into
// its machine, gain (x - ref).
template <typename R, typename Ptr>
__device__ __forceinline__ R sde_rhs(Ptr q, R x, R w, R& inj) {
  const R mu = q[SDE_M0] + x * (q[SDE_M1] + x * q[SDE_M2]);
  R sg, ssp;  // sigma and sigma sigma'
  if (q[SDE_FORM] == R(2)) {
    const R d = x - q[SDE_R];
    const R g = q[SDE_C0] + x * (q[SDE_C1] + x * q[SDE_C2]) + q[SDE_C3] * fabs(d);
    const R sgn = d > R(0) ? R(1) : (d < R(0) ? R(-1) : R(0));
    const R dg = q[SDE_C1] + R(2) * q[SDE_C2] * x + q[SDE_C3] * sgn;
    const bool pos = g > R(0);
    sg = pos ? sqrt(g) : R(0);
    ssp = pos ? R(0.5) * dg : R(0);
  } else {
    sg = q[SDE_C0] + x * (q[SDE_C1] + x * q[SDE_C2]);
    ssp = sg * (q[SDE_C1] + R(2) * q[SDE_C2] * x);
  }
  inj = q[SDE_GAIN] * (x - q[SDE_REF]);
  return mu - q[SDE_K] * ssp + sg * w;
}

// The packed coefficients as a lane reads them.  From memory: the pointer is
// derived again at every stage, so that the compiler streams the machine data
// through scalar loads instead of keeping it live in (spilled) registers across
// stages and steps.  In vector registers, for systems of one or two machines
// (14 or 46 values): their kernels are bound by latency, and a scalar load's
// would be on every stage.
template <typename R>
struct CoefMem {
  const R* p;
  __device__ __forceinline__ cptr<R> stage() const {
    const R* q = p;
    asm volatile("" : "+s"(q));
    return (cptr<R>)q;
  }
};
template <typename R, int N>
struct CoefReg {
  R r[N];
  __device__ __forceinline__ explicit CoefReg(const R* p) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      r[i] = p[i];
      asm volatile("" : "+v"(r[i]));
    }
  }
  __device__ __forceinline__ const R* stage() const { return r; }
};

// Right-hand side of the swing equations + the disturbances in deviation
// form: OU from the packed theta and sigma, or (GEN) the general processes of
// sdeg.  GEN is a separate instantiation so that the OU kernels keep their
// register allocation.
template <typename R, int NG, int PM, bool GEN, typename CF>
__device__ __forceinline__ void swing_rhs(const CF& coef, const R* sdeg, const R wb,
                                          const R (&yd)[NG], const R (&yw)[NG],
                                          const R (&yx)[PM], const R (&wv)[PM], R (&kd)[NG],
                                          R (&kw)[NG], R (&kx)[PM]) {
  constexpr PackLayout L{NG, PM};
  const auto cf = coef.stage();
  // general processes first: their injections feed the machines
  R xin[GEN ? PM : 1];
  if constexpr (GEN) {
    const cptr<R> sq = (cptr<R>)sdeg;
#pragma unroll
    for (int p = 0; p < PM; ++p) kx[p] = sde_rhs<R>(sq + p * kSdeCols, yx[p], wv[p], xin[p]);
  }
  R dc[NG], ds[NG];
  if constexpr (NG <= 2) {
    R sd[NG], omc[NG];
    bool live[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) live[k] = cf[L.c0() + k] != R(0) || cf[L.s0() + k] != R(0);
    rotation_many(yd, live, sd, omc);
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      const R c0 = cf[L.c0() + k], s0 = cf[L.s0() + k];
      dc[k] = -(c0 * omc[k] + s0 * sd[k]);
      ds[k] = c0 * sd[k] - s0 * omc[k];
    }
  } else {
    // the branch-free form: a lane's machines are interleaved by the compiler
    // around the scalar loads of their data
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      R sh, ch;
      sincos_r_nb(yd[k] * R(0.5), sh, ch);
      const R c0 = cf[L.c0() + k], s0 = cf[L.s0() + k];
      const R sd = R(2) * sh * ch;   // sin d
      const R omc = R(2) * sh * sh;  // 1 - cos d
      dc[k] = -(c0 * omc + s0 * sd);
      ds[k] = c0 * sd - s0 * omc;
    }
  }
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    R ir = R(0), ii = R(0);
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      const R yr = cf[L.yre() + i * NG + k];
      const R yi = cf[L.yim() + i * NG + k];
      // complex MAC as four FMAs (no intermediate products)
      ir = fma(yr, dc[k], ir);
      ir = fma(-yi, ds[k], ir);
      ii = fma(yr, ds[k], ii);
      ii = fma(yi, dc[k], ii);
    }
    const R dpe = dc[i] * cf[L.i0r() + i] + ds[i] * cf[L.i0i() + i] +
                  (cf[L.c0() + i] + dc[i]) * ir + (cf[L.s0() + i] + ds[i]) * ii;
    R F = cf[L.res() + i] - dpe - cf[L.dmp() + i] * yw[i];
#pragma unroll
    for (int p = 0; p < PM; ++p) {
      if constexpr (GEN)
        F += cf[L.binc() + i * PM + p] * xin[p];
      else
        F += cf[L.binc() + i * PM + p] * yx[p];
    }
    kd[i] = wb * yw[i];
    kw[i] = F * cf[L.inv2h() + i];
  }
  if constexpr (!GEN) {
#pragma unroll
    for (int p = 0; p < PM; ++p) kx[p] = -cf[L.theta() + p] * yx[p] + cf[L.sigma() + p] * wv[p];
  }
}

// u = sum_v w_v y_v of one trajectory held whole by one lane (absolute angles
// as the outputs store them), FP64.
template <typename R, int NG, int PM>
__device__ __forceinline__ double rrf_u_lane(const IntegArgs<R>& a, double coff, const R (&yd)[NG],
                                             const R (&yw)[NG], const R (&yx)[PM]) {
  const int n = a.n, P = a.P;
  double u = 0.0;  // in output order: angles, speed deviations, processes
#pragma unroll
  for (int i = 0; i < NG; ++i)
    if (i < n) u += a.rrf_w[i] * (a.delta0[i] + (coff + (double)yd[i]));
#pragma unroll
  for (int i = 0; i < NG; ++i)
    if (i < n) u += a.rrf_w[n + i] * (double)yw[i];
#pragma unroll
  for (int p = 0; p < PM; ++p)
    if (p < P) u += a.rrf_w[2 * n + p] * (double)yx[p];
  return u;
}

// Output steps a wave collects before it reduces them: as many as give about
// half the lanes a (step, variable) row each, one where a step has more
// variables than that.  (One machine, 1000 samples, 1000 steps, FP64: 5.74 ms
// with the rows reduced step by step by three lanes; 32 rows, not 64, keep the
// tile at 17 KB, so that nine waves still fit a CU at large N.)
template <int VM>
constexpr int lane_steps() {
  return VM >= 32 ? 1 : 32 / VM;
}

// The outputs of step s into row b of the wave's tile, and of a selected
// sample into its trajectory.
template <typename R, int NG, int PM, int VM>
__device__ __forceinline__ void emit_step(const IntegArgs<R>& a, double (*tile)[VM][65], int b,
                                          int lane, int64_t s, int slot, double coff,
                                          const R (&yd)[NG], const R (&yw)[NG],
                                          const R (&yx)[PM]) {
  const int n = a.n, P = a.P, V = a.V;
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    if (i < n) {
      tile[b][i][lane] = coff + (double)yd[i];
      tile[b][n + i][lane] = (double)yw[i];
    }
  }
#pragma unroll
  for (int p = 0; p < PM; ++p)
    if (p < P) tile[b][2 * n + p][lane] = (double)yx[p];
  if (slot >= 0) {
    double* o = a.traj + ((int64_t)slot * (a.S + 1) + s) * V;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      if (i < n) {
        o[i] = a.delta0[i] + (coff + (double)yd[i]);
        o[n + i] = (double)yw[i];
      }
    }
#pragma unroll
    for (int p = 0; p < PM; ++p)
      if (p < P) o[2 * n + p] = (double)yx[p];
  }
}

// Two-pass statistics of the nb collected steps from s_first on, a lane per
// (step, variable) row of the wave's cnt valid trajectories, each sum in four
// parts over entries j mod 4.
template <typename R, int VM>
__device__ __forceinline__ void reduce_steps(const IntegArgs<R>& a, double (*tile)[VM][65],
                                             int lane, int cnt, int64_t s_first, int nb) {
  const int V = a.V;
  const int64_t S1 = a.S + 1;
  __syncthreads();
  for (int rv = lane; rv < nb * V; rv += 64) {
    const int b = rv / V, v = rv % V;
    const double* row = tile[b][v];
    const double k = row[0];  // the mean as an offset from the first sample: exact for equal ones
    double q0 = 0.0, q1 = 0.0, q2 = 0.0, q3 = 0.0;
    int j = 0;
#pragma unroll 4
    for (; j + 3 < cnt; j += 4) {
      q0 += row[j] - k;
      q1 += row[j + 1] - k;
      q2 += row[j + 2] - k;
      q3 += row[j + 3] - k;
    }
    for (; j < cnt; ++j) q0 += row[j] - k;
    const double mu = k + ((q0 + q1) + (q2 + q3)) / (double)cnt;
    q0 = q1 = q2 = q3 = 0.0;
#pragma unroll 4
    for (j = 0; j + 3 < cnt; j += 4) {
      const double d0 = row[j] - mu, d1 = row[j + 1] - mu, d2 = row[j + 2] - mu, d3 = row[j + 3] - mu;
      q0 = fma(d0, d0, q0);
      q1 = fma(d1, d1, q1);
      q2 = fma(d2, d2, q2);
      q3 = fma(d3, d3, q3);
    }
    for (; j < cnt; ++j) {
      const double d = row[j] - mu;
      q0 = fma(d, d, q0);
    }
    double2* dst = reinterpret_cast<double2*>(a.partial);
    dst[((int64_t)blockIdx.x * S1 + s_first + b) * V + v] = make_double2(mu, (q0 + q1) + (q2 + q3));
  }
  __syncthreads();
}

template <typename R, int NG, int PM, bool GEN = false>
__global__ void __launch_bounds__(64) k_rk4_lane(IntegArgs<R> a) {
  constexpr PackLayout L{NG, PM};
  constexpr int VM = 2 * NG + PM, D = lane_steps<VM>();
  __shared__ double tile[D][VM][65];
  const int lane = threadIdx.x;
  const int64_t gidx = (int64_t)blockIdx.x * 64 + lane;
  const int64_t N = a.N;
  const bool valid = gidx < N;
  const int64_t ns = valid ? gidx : N - 1;
  const int64_t rem = N - (int64_t)blockIdx.x * 64;
  const int cnt = rem < 64 ? (int)rem : 64;
  const int P = a.P;
  const R* __restrict__ cf = a.coef;
  const R* __restrict__ w = a.w;
  using Coef = std::conditional_t<(NG <= 2), CoefReg<R, L.size()>, CoefMem<R>>;
  const Coef coef{cf};
  const int slot = (valid && a.traj_slot) ? a.traj_slot[ns] : -1;

  R yd[NG], yw[NG], yx[PM];
  double coff = 0.0;  // common-angle offset of the trajectory (see IntegArgs::recenter)
  double racc = 0.0;  // the epilogue's RRF sum (see IntegArgs::rrf_w)
  int nbuf = 0;       // steps in the tile, from s_first on
  int64_t s_first = 0;
  if (a.s_begin == 0) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      yd[i] = R(0);
      yw[i] = R(0);
    }
#pragma unroll
    for (int p = 0; p < PM; ++p) yx[p] = cf[L.xi0() + p];
    emit_step<R, NG, PM, VM>(a, tile, 0, lane, 0, slot, coff, yd, yw, yx);
    nbuf = 1;
    if (a.rrf_w) {
      const double u = rrf_u_lane<R, NG, PM>(a, coff, yd, yw, yx);
      racc = 0.5 * u * u;
    }
  } else {
    if (a.rrf_w) racc = a.rrf_acc[ns];
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      yd[i] = a.state[(int64_t)i * a.lanes + gidx];
      yw[i] = a.state[(int64_t)(NG + i) * a.lanes + gidx];
    }
#pragma unroll
    for (int p = 0; p < PM; ++p) yx[p] = a.state[(int64_t)(2 * NG + p) * a.lanes + gidx];
    coff = load_offset(a.state, (int64_t)(2 * NG + PM) * a.lanes + gidx,
                       (int64_t)(2 * NG + PM + 1) * a.lanes + gidx);
  }

  const R dt = a.dt, h2 = a.dt * R(0.5), dt6 = a.dt / R(6), wb = a.wb;
  const R inv_n = R(1) / (R)a.n_ref;
  // KLE path values of the next step are loaded one step ahead.
  R w0[PM], w1[PM], w2[PM];
#pragma unroll
  for (int p = 0; p < PM; ++p) {
    w0[p] = (p < P) ? w[(int64_t)p * N + ns] : R(0);
    w1[p] = (p < P) ? w[((int64_t)1 * P + p) * N + ns] : R(0);
    w2[p] = (p < P) ? w[((int64_t)2 * P + p) * N + ns] : R(0);
  }

  for (int64_t s = a.s_begin; s < a.s_end; ++s) {
    const int64_t cl = 2 * s - a.c_base;
    const bool more = s + 1 < a.s_end;
    R n1[PM], n2[PM];
#pragma unroll
    for (int p = 0; p < PM; ++p) {
      n1[p] = (more && p < P) ? w[((cl + 3) * P + p) * N + ns] : R(0);
      n2[p] = (more && p < P) ? w[((cl + 4) * P + p) * N + ns] : R(0);
    }
    R kd[NG], kw[NG], kx[PM];
    R ad[NG], aw[NG], ax[PM];
    R td[NG], tw[NG], tx[PM];
    // stage 1
    swing_rhs<R, NG, PM, GEN>(coef, GEN ? a.sde : nullptr, wb, yd, yw, yx, w0, kd, kw, kx);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      ad[i] = kd[i]; aw[i] = kw[i];
      td[i] = yd[i] + h2 * kd[i]; tw[i] = yw[i] + h2 * kw[i];
    }
#pragma unroll
    for (int p = 0; p < PM; ++p) { ax[p] = kx[p]; tx[p] = yx[p] + h2 * kx[p]; }
    // stage 2
    swing_rhs<R, NG, PM, GEN>(coef, GEN ? a.sde : nullptr, wb, td, tw, tx, w1, kd, kw, kx);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      ad[i] += R(2) * kd[i]; aw[i] += R(2) * kw[i];
      td[i] = yd[i] + h2 * kd[i]; tw[i] = yw[i] + h2 * kw[i];
    }
#pragma unroll
    for (int p = 0; p < PM; ++p) { ax[p] += R(2) * kx[p]; tx[p] = yx[p] + h2 * kx[p]; }
    // stage 3
    swing_rhs<R, NG, PM, GEN>(coef, GEN ? a.sde : nullptr, wb, td, tw, tx, w1, kd, kw, kx);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      ad[i] += R(2) * kd[i]; aw[i] += R(2) * kw[i];
      td[i] = yd[i] + dt * kd[i]; tw[i] = yw[i] + dt * kw[i];
    }
#pragma unroll
    for (int p = 0; p < PM; ++p) { ax[p] += R(2) * kx[p]; tx[p] = yx[p] + dt * kx[p]; }
    // stage 4
    swing_rhs<R, NG, PM, GEN>(coef, GEN ? a.sde : nullptr, wb, td, tw, tx, w2, kd, kw, kx);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      yd[i] += dt6 * (ad[i] + kd[i]);
      yw[i] += dt6 * (aw[i] + kw[i]);
    }
#pragma unroll
    for (int p = 0; p < PM; ++p) {
      yx[p] += dt6 * (ax[p] + kx[p]);
      w0[p] = w2[p];
      w1[p] = n1[p];
      w2[p] = n2[p];
    }
    if (a.recenter) {  // move the mean angle of the machines in service into the offset
      R sum = R(0);
#pragma unroll
      for (int i = 0; i < NG; ++i)
        if (i < a.n && (cf[L.c0() + i] != R(0) || cf[L.s0() + i] != R(0))) sum += yd[i];
      const R ref = sum * inv_n;
      coff += (double)ref;
#pragma unroll
      for (int i = 0; i < NG; ++i) yd[i] -= ref;
    }
    if (nbuf == D) {
      reduce_steps<R, VM>(a, tile, lane, cnt, s_first, nbuf);
      nbuf = 0;
    }
    if (nbuf == 0) s_first = s + 1;
    emit_step<R, NG, PM, VM>(a, tile, D == 1 ? 0 : nbuf, lane, s + 1, slot, coff, yd, yw, yx);
    ++nbuf;
    if (a.rrf_w) {
      const double u = rrf_u_lane<R, NG, PM>(a, coff, yd, yw, yx);
      racc += (s + 1 == a.S ? 0.5 : 1.0) * u * u;
    }
  }
  reduce_steps<R, VM>(a, tile, lane, cnt, s_first, nbuf);
  if (a.rrf_w && valid) {
    a.rrf_acc[gidx] = racc;
    if (a.s_end == a.S) a.rrf[gidx] = sqrt(racc / (double)a.S);
  }

#pragma unroll
  for (int i = 0; i < NG; ++i) {
    a.state[(int64_t)i * a.lanes + gidx] = yd[i];
    a.state[(int64_t)(NG + i) * a.lanes + gidx] = yw[i];
  }
#pragma unroll
  for (int p = 0; p < PM; ++p) a.state[(int64_t)(2 * NG + p) * a.lanes + gidx] = yx[p];
  store_offset(a.state, (int64_t)(2 * NG + PM) * a.lanes + gidx,
               (int64_t)(2 * NG + PM + 1) * a.lanes + gidx, coff);

  if (a.s_end == a.S && valid) {
    bool bad = !isfinite(coff);
#pragma unroll
    for (int i = 0; i < NG; ++i) bad |= !isfinite(yd[i]) || !isfinite(yw[i]);
#pragma unroll
    for (int p = 0; p < PM; ++p) bad |= !isfinite(yx[p]);
    if (bad) {
      atomicAdd(a.nonfinite, 1ULL);
      atomicMin(a.first_bad, (long long)gidx);
    }
  }
}


// ---------------------------------------------------------------------------
// Group variant: L lanes share one trajectory (any L <= 64; a wave holds
// floor(64/L) trajectories and leaves the remaining lanes idle), lane g owns
// the G = ceil(NG/L) machines g*G .. g*G+G-1 and the rows of Y for them (held
// in registers, read once).  Twice per step (four times in the lean form) each lane
// rotates its own machines for the coming stages, the pairs of a trajectory are
// exchanged through LDS (the lanes of a trajectory are in one wave, whose LDS
// operations complete in order, so only a compiler-level wavefront fence is needed),
// and each lane forms the network sums of its rows.  A disturbance process is
// integrated by one lane (group_run says which).  A workgroup of WPB waves reduces the
// statistics of its trajectories over several collected steps at once.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// *p, the same for all lanes, into scalar registers
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  struct Words {
    int w[sizeof(T) / 4];
  };
  const Words* s = reinterpret_cast<const Words*>(p);
  Words v;
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 4; ++i) v.w[i] = __builtin_amdgcn_readfirstlane(s->w[i]);
  return __builtin_bit_cast(T, v);
}

template <typename R> struct vec2;
template <> struct vec2<double> { using type = double2; };
template <> struct vec2<float> { using type = float2; };

// Form of the network product of the group and team kernels.  FP64: rotated
// (PackLayout), which saves the turn by E0 and the products with it.  FP32:
// plain.  There the rounding of the coefficients is systematic over all samples,
// and rounding Z_ik / 2H_i and Z_ki / 2H_k on their own breaks the balance
// of the two machines' exchange that Y_ik = Y_ki keeps: the common angle drifts
// (45 machines, 19 s: mean off by 1.9e-6 rotated, 5e-7 plain; 6 machines: variance
// by 5.7e-6 and 3.6e-6).
template <typename R>
__host__ __device__ constexpr bool rotated_form() {
  return sizeof(R) == 8;
}

// The group integrator in its lean form: four exchanges per step, a stage each,
// instead of two, and the processes always through the exchange row.  About forty
// registers less, for the systems whose rows of Y leave no room for them (a spilled
// row comes back in every stage).  us per step, 4000 samples, with two exchanges / lean:
// FP64 14 machines 4.4 / 2.1, 20 machines 26 / 16, 45 machines 247 / 145; FP32 20 machines
// 2.6 / 2.9, 30 machines 3.8 / 3.5, general processes 17.6 / 3.6, 45 machines 102 / 25.
template <typename R, int NG>
__host__ __device__ constexpr bool lean_form() {
  return sizeof(R) == 8 ? NG >= 16 : NG >= 32;
}

// A step's change of an angle from the weighted sum su of its stage speeds, dt / 6 w_b su.
// FP32 takes the product with w_b first: the rounding of dt / 6 w_b to one constant is the
// same in every step and shifts the machines' frequency against the speeds (dt = 5 ms:
// the error of the variances over systems of 3 to 24 machines 7 % above, now the same as,
// that of a kernel that forms every stage's w_b u).
__device__ __forceinline__ float angle_step(float dt6, float wb, float su) { return dt6 * (wb * su); }
__device__ __forceinline__ double angle_step(double dt6, double wb, double su) { return dt6 * wb * su; }

// (1 - cos d, sin d) turned by E0: dE = E0 (e^{j d} - 1) = -omc + j sd
template <typename R>
__device__ __forceinline__ void turn(R e0r, R e0i, R& omc, R& sd) {
  const R o = fma(e0i, sd, e0r * omc);
  sd = fma(e0r, sd, -e0i * omc);
  omc = o;
}

// Sizes of one group variant and the LDS it needs: the statistics tile (the
// values of up to D consecutive output steps, reduced together with two
// workgroup barriers per D steps), the exchange rows (NGP machine slots and PM
// process slots per trajectory; row TB is scratch for idle lanes) and the
// non-finite flags.
template <typename R, int NG, int PM, int L, int WPB, int D>
struct GroupShape {
  using R2 = typename vec2<R>::type;
  static constexpr int G = (NG + L - 1) / L;   // machines per lane
  static constexpr int PQ = (PM + L - 1) / L;  // processes per lane
  static constexpr int NGP = G * L;            // padded machine slots per trajectory
  static constexpr int XW = NGP + PM + 1;      // exchange row width (R2 entries)
  static constexpr int TW = 64 / L;            // trajectories per wave
  static constexpr int TB = TW * WPB;          // trajectories per workgroup
  static constexpr int VM = 2 * NG + PM;
  static constexpr size_t tile_bytes = (size_t)D * VM * (TB + 1) * sizeof(double);
  static constexpr size_t xch_bytes = (size_t)2 * (TB + 1) * XW * sizeof(R2);  // two stages
  static constexpr size_t rrf_off = tile_bytes + xch_bytes;  // weights and offsets [2][VM]
  static constexpr size_t bad_off = rrf_off + (size_t)2 * VM * sizeof(double);
  static constexpr size_t lds_bytes = bad_off + (TB + 1) * sizeof(int);
};

// Mean and sum of squared deviations of row[0, cnt) (cnt >= 1) in one pass
// over LDS: with the shift k = row[0] and d = x - k, mean = k + S1/cnt
// and M2 = S2 - S1^2/cnt (S1, S2 the sums of d and d^2, each in four partial
// sums over entries j mod 4, added in a fixed order).  The shift is one of the
// samples, so (mean - k)^2 <= (cnt - 1) M2 / cnt and the subtraction loses at
// most a factor cnt of relative accuracy (about 1e-14 here); equal entries
// give M2 = 0 exactly.
__device__ __forceinline__ void row_stats(const double* row, int cnt, double& mu, double& m2) {
  const double k = row[0];
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  double q0 = 0.0, q1 = 0.0, q2 = 0.0, q3 = 0.0;
  int j = 0;
#pragma unroll 2
  for (; j + 3 < cnt; j += 4) {
    const double d0 = row[j] - k, d1 = row[j + 1] - k, d2 = row[j + 2] - k, d3 = row[j + 3] - k;
    s0 += d0; s1 += d1; s2 += d2; s3 += d3;
    q0 = fma(d0, d0, q0); q1 = fma(d1, d1, q1); q2 = fma(d2, d2, q2); q3 = fma(d3, d3, q3);
  }
  if (j < cnt) { const double d = row[j] - k; s0 += d; q0 = fma(d, d, q0); }
  if (j + 1 < cnt) { const double d = row[j + 1] - k; s1 += d; q1 = fma(d, d, q1); }
  if (j + 2 < cnt) { const double d = row[j + 2] - k; s2 += d; q2 = fma(d, d, q2); }
  const double S1 = (s0 + s1) + (s2 + s3), S2 = (q0 + q1) + (q2 + q3);
  const double dm = S1 / (double)cnt;
  mu = k + dm;
  m2 = fma(-S1, dm, S2);
}

// Where a group run leaves its statistics: rows[(s)*V + v] = (mean, M2) of the
// group's samples; prev > 0 means the rows already hold the statistics of prev
// earlier samples, and the group's are merged in with Chan's update (a fixed
// order, so results do not depend on scheduling).
struct GroupStats {
  double2* rows;
  int64_t prev;
};

// One workgroup integrates trajectories tile*TB .. tile*TB + TB - 1 of a
// scenario over the steps [s_begin, s_end) of a.  Lane g of a trajectory owns
// machines g*G .. g*G+G-1 (rows of Y in registers); per stage the lanes exchange
// the rotated EMF deviations of their machines through LDS.  keep_state stores
// the state for a following chunk.  GEN: the processes are the general Ito
// processes of a.sde.
//
// Processes: with one machine per lane and at most one process at a machine (and not in
// the lean form), the
// lane of the machine owns its process and adds the injection itself (no exchange:
// the wave reads ten pairs per stage instead of fourteen values for ten machines
// and four process slots, and drops the product with the 0/1 injection matrix);
// else lane g owns processes g, g + L, ... and publishes the injected powers in
// the exchange row.  Which of the two holds is the same for all waves and chunks:
// it comes from the packed owner machines, which an event leaves alone.
template <typename R, int NG, int PM, int L, int WPB, int D, bool GEN = false, bool LEAN = lean_form<R, NG>()>
__device__ __forceinline__ void group_run(const IntegArgs<R>& a, int64_t tile,
                                          unsigned char* lds, GroupStats st, bool keep_state) {
  using Sh = GroupShape<R, NG, PM, L, WPB, D>;
  using R2 = typename Sh::R2;
  constexpr PackLayout Lp{NG, PM};
  constexpr int G = Sh::G, PQ = Sh::PQ, NGP = Sh::NGP, XW = Sh::XW, TW = Sh::TW, TB = Sh::TB,
                VM = Sh::VM;
  double (*tile_buf)[VM][TB + 1] = reinterpret_cast<double (*)[VM][TB + 1]>(lds);
  R2 (*xch)[TB + 1][XW] = reinterpret_cast<R2 (*)[TB + 1][XW]>(lds + Sh::tile_bytes);
  double* rrf_l = reinterpret_cast<double*>(lds + Sh::rrf_off);
  int* bad_t = reinterpret_cast<int*>(lds + Sh::bad_off);
  // opaque, so that a persistent kernel's tile loop does not keep every address of
  // the set-up below in registers
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wv = tid >> 6, ln = tid & 63;
  const bool lane_on = ln < TW * L;
  const int tl = lane_on ? wv * TW + ln / L : TB;
  const int g = lane_on ? ln % L : 0;
  const int64_t traj = tile * TB + tl;
  const int64_t N = a.N;
  const bool valid = lane_on && traj < N;
  const int64_t ns = valid ? traj : N - 1;
  const int64_t rem = N - tile * TB;
  const int cnt = rem < TB ? (int)rem : TB;
  const int n = a.n, P = a.P, V = a.V;
  const R* __restrict__ cf = a.coef;
  const R* __restrict__ w = a.w;
  const int slot = (valid && a.traj_slot) ? a.traj_slot[ns] : -1;

  // per-lane machine data (PackLayout): FP64 rotated, rows of Z, J, res, D; FP32
  // plain, rows of Y, I0, res, D, E0 and 1/2H
  constexpr bool ROT = rotated_form<R>();
  R zr[G][NG], zi[G][NG], jr[G], ji[G], res[G], dmp[G], e0r[G], e0i[G], inv2h[G];
  bool live[G];
  int live_mask[G];
#pragma unroll
  for (int q = 0; q < G; ++q) {
    const int i = g * G + q;
    const bool on = i < NG;
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      zr[q][k] = on ? cf[Lp.yre() + i * NG + k] : R(0);
      zi[q][k] = on ? cf[Lp.yim() + i * NG + k] : R(0);
    }
    jr[q] = on ? cf[Lp.i0r() + i] : R(0);
    ji[q] = on ? cf[Lp.i0i() + i] : R(0);
    res[q] = on ? cf[Lp.res() + i] : R(0);
    dmp[q] = on ? cf[Lp.dmp() + i] : R(0);
    e0r[q] = ROT ? R(1) : (on ? cf[Lp.c0() + i] : R(0));
    e0i[q] = ROT ? R(0) : (on ? cf[Lp.s0() + i] : R(0));
    inv2h[q] = ROT ? R(1) : (on ? cf[Lp.inv2h() + i] : R(0));
    // in service: the machine has an EMF
    live[q] = lane_on && on && (cf[Lp.c0() + i] != R(0) || cf[Lp.s0() + i] != R(0));
    live_mask[q] = lane_mask(live[q]);
  }

  // my processes: pid[r], or none (PM)
  int pid[PQ];
  bool local = false;
  constexpr bool kLocal = G == 1 && !LEAN;
#pragma unroll
  for (int r = 0; r < PQ; ++r) pid[r] = lane_on && g + L * r < P ? g + L * r : PM;
  if constexpr (kLocal) {
    int mine = PM, n_mine = 0;
#pragma unroll
    for (int p = PM - 1; p >= 0; --p)
      if (lane_on && p < P && (int)cf[Lp.owner() + p] == g) {
        mine = p;
        ++n_mine;
      }
    local = __builtin_amdgcn_ballot_w64(n_mine > 1) == 0;
    if (local) {
      pid[0] = mine;
#pragma unroll
      for (int r = 1; r < PQ; ++r) pid[r] = PM;
    }
  }
  R theta[PQ], sigma[PQ];
  bool own[PQ];
  int own_mask[PQ];
  int64_t wofs[PQ];
  R sde[GEN ? PQ : 1][kSdeCols];  // GEN: my processes' rows (zero: none)
  bool root = false, poly = false;  // GEN: some lane has a process of the form
#pragma unroll
  for (int r = 0; r < PQ; ++r) {
    own[r] = pid[r] < PM;
    own_mask[r] = lane_mask(own[r]);
    theta[r] = !GEN && own[r] ? cf[Lp.theta() + pid[r]] : R(0);
    sigma[r] = !GEN && own[r] ? cf[Lp.sigma() + pid[r]] : R(0);
    wofs[r] = own[r] ? (int64_t)pid[r] * N + ns : 0;
    if constexpr (GEN) {
#pragma unroll
      for (int c = 0; c < kSdeCols; ++c) sde[r][c] = own[r] ? a.sde[pid[r] * kSdeCols + c] : R(0);
      root = root || sde[r][SDE_FORM] == R(2);
      poly = poly || sde[r][SDE_FORM] == R(1);
    }
  }
  if constexpr (GEN) {
    root = __builtin_amdgcn_ballot_w64(root) != 0;
    poly = __builtin_amdgcn_ballot_w64(poly) != 0;
  }
  // injection: local, the factor of my process at my machine; else the
  // machines' rows of the injection matrix
  R binl = R(0), binc[G][PM];
#pragma unroll
  for (int q = 0; q < G; ++q)
#pragma unroll
    for (int p = 0; p < PM; ++p) {
      const int i = g * G + q;
      binc[q][p] = i < NG ? cf[Lp.binc() + i * PM + p] : R(0);
      if (kLocal && local && p == pid[0]) binl = binc[q][p];
    }

  // the process slots p >= P of my trajectory's exchange rows stay zero
  auto clear_slots = [&]() {
    if (g == 0) {
#pragma unroll
      for (int p = 0; p < PM; ++p) xch[0][tl][NGP + p] = xch[1][tl][NGP + p] = R2{R(0), R(0)};
    }
    wave_lds_sync();
  };
  clear_slots();

  // RK4 of the swing equations in two exchanges per step: the angles of stages
  // 1 and 2 are known at the start of the step (an angle's derivative is its
  // speed), those of stages 3 and 4 once the accelerations of 1 and 2 are.  So
  // stages 1 and 2, then 3 and 4, share one rotation, one exchange and one pass
  // over the rows of Y.
  //
  // (The lean form takes a stage at a time: H = 1.)
  //
  // Network part of H stages at angles d[h]: rotation, exchange
  // and, per machine, sum_k Z_ik eps_k (cr, ci); in the plain form sum_k Y_ik dE_k
  // of the rotated EMFs' deviations dE = -omc + j sd, omc and sd then turned by E0.
  constexpr int H = LEAN ? 1 : 2;
  R sd[H][G], omc[H][G], cr[H][G], ci[H][G];
  auto network = [&](const R (&d)[H][G], const R (&pub)[H][PQ]) {
    rotation_stages<R, H, G>(d, live, live_mask, sd, omc);
    if constexpr (!ROT) {
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int q = 0; q < G; ++q) turn(e0r[q], e0i[q], omc[h][q], sd[h][q]);
    }
#pragma unroll
    for (int h = 0; h < H; ++h) {
#pragma unroll
      for (int q = 0; q < G; ++q) {
        // a machine without EMF has a zero column of Z and turns by zero
        xch[h][tl][g * G + q] = R2{omc[h][q], sd[h][q]};
        cr[h][q] = ci[h][q] = R(0);
      }
      if (!local) {
#pragma unroll
        for (int r = 0; r < PQ; ++r)
          if (own[r]) xch[h][tl][NGP + pid[r]] = R2{pub[h][r], R(0)};
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      // keep at most 8 exchange loads in flight: bounds the registers the
      // scheduler would otherwise spend hoisting all of them
      if ((k & 3) == 0 && k > 0) asm volatile("" ::: "memory");
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const R2 e = xch[h][tl][k];  // eps = -e.x + j e.y
#pragma unroll
        for (int q = 0; q < G; ++q) {
          // complex MAC as four FMAs; a dependent FMA issues as soon as the
          // pipe is free, so one chain per component is enough
          cr[h][q] = fma(-zr[q][k], e.x, cr[h][q]);
          ci[h][q] = fma(-zi[q][k], e.x, ci[h][q]);
          cr[h][q] = fma(-zi[q][k], e.y, cr[h][q]);
          ci[h][q] = fma(zr[q][k], e.y, ci[h][q]);
        }
      }
    }
    if (local) wave_lds_sync();
  };
  // injected powers of my machines in stage h
  auto injection = [&](int h, const R (&pub)[PQ], R (&inj)[G]) {
    if (kLocal && local) {  // wave-uniform
      inj[0] = binl * pub[0];
      return;
    }
#pragma unroll
    for (int q = 0; q < G; ++q) inj[q] = R(0);
    // every process slot, the padding ones included (zero, as their columns
    // of binc)
#pragma unroll
    for (int p = 0; p < PM; ++p) {
      const R xp = xch[h][tl][NGP + p].x;
#pragma unroll
      for (int q = 0; q < G; ++q) inj[q] += binc[q][p] * xp;
    }
    wave_lds_sync();
  };
  // accelerations of my machines in stage h at speeds u
  auto accel = [&](int h, const R (&u)[G], const R (&inj)[G], R (&kw)[G]) {
#pragma unroll
    for (int q = 0; q < G; ++q) {
      R F = res[q] - dmp[q] * u[q] + inj[q];
      F = fma(omc[h][q], jr[q], F);
      F = fma(-sd[h][q], ji[q], F);
      if constexpr (ROT) {
        F = fma(omc[h][q] - R(1), cr[h][q], F);
        kw[q] = fma(-sd[h][q], ci[h][q], F);
      } else {
        F = fma(omc[h][q] - e0r[q], cr[h][q], F);
        F = fma(-(e0i[q] + sd[h][q]), ci[h][q], F);
        kw[q] = F * inv2h[q];
      }
    }
  };
  // derivative of my process r at x with path value wv, and what it injects
  auto rate = [&](int r, R x, R wv) {
    if constexpr (GEN)
      return sde_rate(sde[r], x, wv, root, poly);
    else
      return sigma[r] * wv - theta[r] * x;
  };
  auto power = [&](int r, R x) {
    if constexpr (GEN)
      return sde[r][SDE_GAIN] * (x - sde[r][SDE_REF]);
    else
      return x;
  };

  // RRF sum of trajectory tid of this tile (threads tid < TB; see IntegArgs::rrf_w)
  double racc = 0.0;
  if (a.rrf_w) {
    if (a.s_begin > 0 && tid < cnt) racc = a.rrf_acc[tile * TB + tid];
    // the weights and the outputs' offsets, read by every term of every step
    // (visible after the first flush's barrier)
    for (int v = tid; v < V; v += 64 * WPB) {
      rrf_l[v] = a.rrf_w[v];
      rrf_l[VM + v] = v < n ? a.delta0[v] : 0.0;
    }
  }
  // Reduce the buffered steps [s_first, s_first + nb): thread q of the
  // workgroup takes rows (step, variable) q, q + 64 WPB, ...
  auto flush = [&](int64_t s_first, int nb) {
    __syncthreads();
    for (int rv = tid; rv < nb * V; rv += 64 * WPB) {
      const int b = rv / V, v = rv % V;
      double mu, m2;
      row_stats(tile_buf[b][v], cnt, mu, m2);
      double2* dst = st.rows + (s_first + b) * V + v;
      if (st.prev == 0) {
        *dst = make_double2(mu, m2);
      } else {
        const double2 old = *dst;
        const double na = (double)st.prev, nb2 = (double)cnt, tot = na + nb2;
        const double dl = mu - old.x;
        *dst = make_double2(old.x + dl * (nb2 / tot), old.y + m2 + dl * dl * (na * nb2 / tot));
      }
    }
    // the epilogue's RRF: a thread per (buffered step, trajectory) forms u and leaves
    // h u^2 in its trajectory's exchange row (free between steps), then thread j
    // adds trajectory j's in step order
    if (a.rrf_w) {
      static_assert((size_t)D * TB * sizeof(double) <= Sh::xch_bytes, "room for the RRF terms");
      double* term = reinterpret_cast<double*>(lds + Sh::tile_bytes);
      for (int q = tid; q < nb * TB; q += 64 * WPB) {
        const int b = q / TB, j = q - b * TB;
        const int64_t s = s_first + b;
        double u = 0.0;
#pragma unroll 4
        for (int v = 0; v < V; ++v) u += rrf_l[v] * (rrf_l[VM + v] + tile_buf[b][v][j]);
        term[q] = (s == 0 || s == a.S ? 0.5 : 1.0) * u * u;
      }
      __syncthreads();
      if (tid < cnt)
        for (int b = 0; b < nb; ++b) racc += term[b * TB + tid];
      __syncthreads();
      clear_slots();
    }
    __syncthreads();
  };
  int nbuf = 0;
  int64_t s_first = 0;
  double coff = 0.0;  // common-angle offset of my trajectory (see IntegArgs::recenter)
  // Where my outputs go in a buffered step's rows; machines and processes that do
  // not exist write the padding column TB (idle lanes are in it anyway), so
  // that no lane branches.
  int od[G], ow[G], ox[PQ];
#pragma unroll
  for (int q = 0; q < G; ++q) {
    const int i = g * G + q;
    od[q] = i < n ? i * (TB + 1) + tl : TB;
    ow[q] = i < n ? (n + i) * (TB + 1) + tl : TB;
  }
#pragma unroll
  for (int r = 0; r < PQ; ++r) ox[r] = own[r] ? (2 * n + pid[r]) * (TB + 1) + tl : TB;
  const bool traced = __builtin_amdgcn_ballot_w64(slot >= 0) != 0;  // some lane stores a trajectory
  auto emit = [&](int64_t s, const R (&yd)[G], const R (&yw)[G], const R (&yx)[PQ]) {
    if (nbuf == 0) s_first = s;
    double* tb = &tile_buf[nbuf][0][0];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      tb[od[q]] = coff + (double)yd[q];
      tb[ow[q]] = (double)yw[q];
    }
#pragma unroll
    for (int r = 0; r < PQ; ++r) tb[ox[r]] = (double)yx[r];
    if (traced && slot >= 0) {
      // every lane of a selected trajectory writes its own outputs
      double* o = a.traj + ((int64_t)slot * (a.S + 1) + s) * V;
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const int i = g * G + q;
        if (i < n) {
          o[i] = a.delta0[i] + (coff + (double)yd[q]);
          o[n + i] = (double)yw[q];
        }
      }
#pragma unroll
      for (int r = 0; r < PQ; ++r)
        if (own[r]) o[2 * n + pid[r]] = (double)yx[r];
    }
    if (++nbuf == D) {
      flush(s_first, nbuf);
      nbuf = 0;
    }
  };

  R yd[G], yw[G], yx[PQ];
  const int64_t lane_id = tile * 64 * WPB + tid;
  if (a.s_begin == 0) {
#pragma unroll
    for (int q = 0; q < G; ++q) { yd[q] = R(0); yw[q] = R(0); }
#pragma unroll
    for (int r = 0; r < PQ; ++r) yx[r] = own[r] ? cf[Lp.xi0() + pid[r]] : R(0);
    emit(0, yd, yw, yx);
  } else {
#pragma unroll
    for (int q = 0; q < G; ++q) {
      yd[q] = a.state[(int64_t)q * a.lanes + lane_id];
      yw[q] = a.state[(int64_t)(G + q) * a.lanes + lane_id];
    }
#pragma unroll
    for (int r = 0; r < PQ; ++r) yx[r] = a.state[(int64_t)(2 * G + r) * a.lanes + lane_id];
    coff = load_offset(a.state, (int64_t)(2 * G + PQ) * a.lanes + lane_id,
                       (int64_t)(2 * G + PQ + 1) * a.lanes + lane_id);
  }

  const R dt = a.dt, h2 = a.dt * R(0.5), dt6 = a.dt / R(6);
  const R hw2 = h2 * a.wb, hw = dt * a.wb;
  const R inv_n = R(1) / (R)a.n_ref;
  const int64_t colstride = (int64_t)P * N;
  // KLE path values of my processes: the two new stage columns of a step are
  // loaded two steps ahead (a step of a lone wave is shorter than the latency
  // of memory).
  // A lane without a process loads the first process's path of the first sample
  // and masks it (its sigma is zero, that path may not be finite), the last steps read
  // the last columns again: no lane branches.
  R w0[PQ], w1[PQ], w2[PQ], n1[PQ], n2[PQ];
  auto column = [&](int64_t s) {  // first column of step s of this chunk
    return (2 * (s < a.s_end ? s : a.s_end - 1) - a.c_base) * colstride;
  };
  {
    const int64_t c1 = column(a.s_begin + 1);
#pragma unroll
    for (int r = 0; r < PQ; ++r) {
      w0[r] = masked(own_mask[r], w[wofs[r]]);
      w1[r] = masked(own_mask[r], w[colstride + wofs[r]]);
      w2[r] = masked(own_mask[r], w[2 * colstride + wofs[r]]);
      n1[r] = w[c1 + colstride + wofs[r]];
      n2[r] = w[c1 + 2 * colstride + wofs[r]];
    }
  }
  for (int64_t s = a.s_begin; s < a.s_end; ++s) {
    const int64_t c2 = column(s + 2);
    R m1[PQ], m2[PQ];
#pragma unroll
    for (int r = 0; r < PQ; ++r) {
      m1[r] = w[c2 + colstride + wofs[r]];
      m2[r] = w[c2 + 2 * colstride + wofs[r]];
    }
    // the four stage values of my processes (they do not see the machines)
    R pub[4][PQ];
#pragma unroll
    for (int r = 0; r < PQ; ++r) {
      const R x1 = yx[r], k1 = rate(r, x1, w0[r]);
      const R x2 = x1 + h2 * k1, k2 = rate(r, x2, w1[r]);
      const R x3 = x1 + h2 * k2, k3 = rate(r, x3, w1[r]);
      const R x4 = x1 + dt * k3, k4 = rate(r, x4, w2[r]);
      pub[0][r] = power(r, x1);
      pub[1][r] = power(r, x2);
      pub[2][r] = power(r, x3);
      pub[3][r] = power(r, x4);
      yx[r] = x1 + dt6 * (((k1 + R(2) * k2) + R(2) * k3) + k4);
      w0[r] = w2[r];
      w1[r] = masked(own_mask[r], n1[r]);
      w2[r] = masked(own_mask[r], n2[r]);
      n1[r] = m1[r];
      n2[r] = m2[r];
    }
    // the angles' derivatives are w_b times the stage speeds: their sum runs
    // over the speeds, and w_b sits in the step constants
    R d[H][G], u[2][G], kw[G], inj[G], su[G], sa[G];
    using Pub = const R (*)[H][PQ];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      d[0][q] = yd[q];
      if constexpr (H == 2) d[1][q] = yd[q] + hw2 * yw[q];
    }
    network(d, *reinterpret_cast<Pub>(&pub[0]));
    injection(0, pub[0], inj);
    accel(0, yw, inj, kw);
#pragma unroll
    for (int q = 0; q < G; ++q) {
      if constexpr (H == 1) d[0][q] = yd[q] + hw2 * yw[q];
      u[0][q] = yw[q] + h2 * kw[q];
      su[q] = yw[q] + R(2) * u[0][q];
      sa[q] = kw[q];
    }
    if constexpr (H == 1) network(d, *reinterpret_cast<Pub>(&pub[1]));
    injection(H - 1, pub[1], inj);
    accel(H - 1, u[0], inj, kw);
#pragma unroll
    for (int q = 0; q < G; ++q) {
      d[0][q] = yd[q] + hw2 * u[0][q];
      u[1][q] = yw[q] + h2 * kw[q];
      su[q] += R(2) * u[1][q];
      sa[q] += R(2) * kw[q];
      if constexpr (H == 2) d[1][q] = yd[q] + hw * u[1][q];
    }
    network(d, *reinterpret_cast<Pub>(&pub[2]));
    injection(0, pub[2], inj);
    accel(0, u[1], inj, kw);
#pragma unroll
    for (int q = 0; q < G; ++q) {
      if constexpr (H == 1) d[0][q] = yd[q] + hw * u[1][q];
      u[0][q] = yw[q] + dt * kw[q];
      su[q] += u[0][q];
      sa[q] += R(2) * kw[q];
    }
    if constexpr (H == 1) network(d, *reinterpret_cast<Pub>(&pub[3]));
    injection(H - 1, pub[3], inj);
    accel(H - 1, u[0], inj, kw);
#pragma unroll
    for (int q = 0; q < G; ++q) {
      yd[q] += angle_step(dt6, a.wb, su[q]);
      yw[q] += dt6 * (sa[q] + kw[q]);
    }
    if (a.recenter && ((s + 1) & 7) == 0) {
      // every eighth step (of the absolute step count, so time chunks keep the
      // bits; the common angle moves by milliradians in between):
      // the mean angle of the trajectory's machines in service (a tripped
      // machine has no EMF): each lane's sum over its machines through the
      // exchange row (free again: the last stage's reads ended with a wave
      // fence), added in lane order by every lane of the trajectory (the same
      // bits in each), then taken out of every angle
      R part = R(0);
#pragma unroll
      for (int q = 0; q < G; ++q)
        if (live[q]) part += yd[q];
      xch[0][tl][g] = R2{part, R(0)};
      wave_lds_sync();
      R sum = R(0);
      for (int k = 0; k < L; ++k) sum += xch[0][tl][k].x;
      wave_lds_sync();
      const R ref = sum * inv_n;
      coff += (double)ref;
#pragma unroll
      for (int q = 0; q < G; ++q)  // padding machines stay at rest
        if (g * G + q < n) yd[q] -= ref;
    }
    emit(s + 1, yd, yw, yx);
  }

  if (nbuf > 0) flush(s_first, nbuf);  // nbuf is uniform over the workgroup
  if (a.rrf_w && tid < cnt) {
    a.rrf_acc[tile * TB + tid] = racc;
    if (a.s_end == a.S) a.rrf[tile * TB + tid] = sqrt(racc / (double)a.S);
  }

  if (keep_state) {
#pragma unroll
    for (int q = 0; q < G; ++q) {
      a.state[(int64_t)q * a.lanes + lane_id] = yd[q];
      a.state[(int64_t)(G + q) * a.lanes + lane_id] = yw[q];
    }
#pragma unroll
    for (int r = 0; r < PQ; ++r) a.state[(int64_t)(2 * G + r) * a.lanes + lane_id] = yx[r];
    store_offset(a.state, (int64_t)(2 * G + PQ) * a.lanes + lane_id,
                 (int64_t)(2 * G + PQ + 1) * a.lanes + lane_id, coff);
  }

  if (a.s_end == a.S) {  // uniform over the workgroup: the barriers below are safe
    bool bad = !isfinite(coff);
#pragma unroll
    for (int q = 0; q < G; ++q) bad |= !isfinite(yd[q]) || !isfinite(yw[q]);
#pragma unroll
    for (int r = 0; r < PQ; ++r) bad |= !isfinite(yx[r]);
    // one count per trajectory: the lanes of a trajectory combine through LDS
    if (lane_on && g == 0) bad_t[tl] = 0;
    __syncthreads();
    if (lane_on && bad) bad_t[tl] = 1;
    __syncthreads();
    if (valid && g == 0 && bad_t[tl] != 0) {
      atomicAdd(a.nonfinite, 1ULL);
      atomicMin(a.first_bad, (long long)traj);
    }
    __syncthreads();  // the flags may be reused by the workgroup's next run
  }
}

// At least two waves per SIMD (at most 256 registers per lane, VGPRs and
// AGPRs together): left to itself the compiler spends all 256 VGPRs plus a
// few AGPRs on the larger variants and drops them to one wave per SIMD.
#ifndef FMC_GROUP_MIN_WAVES
#define FMC_GROUP_MIN_WAVES 2
#endif
template <typename R, int NG, int PM, int L, int WPB>
__global__ void __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(FMC_GROUP_MIN_WAVES)))
k_rk4_group(IntegArgs<R> a) {
  constexpr int D = WPB == 1 ? 4 : 8;
  using Sh = GroupShape<R, NG, PM, L, WPB, D>;
  __shared__ __attribute__((aligned(16))) unsigned char lds[Sh::lds_bytes];
  GroupStats st{reinterpret_cast<double2*>(a.partial) + (int64_t)blockIdx.x * (a.S + 1) * a.V, 0};
  group_run<R, NG, PM, L, WPB, D>(a, blockIdx.x, lds, st, true);
}

template <typename R, int NG, int PM, int L, int WPB, bool GEN>
__global__ void __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(3)))
k_rk4_group_lean(IntegArgs<R> a) {
  constexpr int D = WPB == 1 ? 4 : 8;
  using Sh = GroupShape<R, NG, PM, L, WPB, D>;
  __shared__ __attribute__((aligned(16))) unsigned char lds[Sh::lds_bytes];
  GroupStats st{reinterpret_cast<double2*>(a.partial) + (int64_t)blockIdx.x * (a.S + 1) * a.V, 0};
  group_run<R, NG, PM, L, WPB, D, GEN, true>(a, blockIdx.x, lds, st, true);
}

// 16 machines in FP32 fit three waves per SIMD in the lean form, two in the other: a
// launch of more than two and at most three waves per SIMD takes the lean one (returns
// whether it did).  us per step, 14 machines, general processes, lean / other: 8000
// samples (2.0 waves) 2.4 / 2.3, 8300 3.1 / 3.7, 12000 (2.9) 3.1 / 3.8, 16000 4.9 / 4.6,
// 24000 6.9 / 6.9.
template <typename R, int NG, int PM, int L, int WPB, bool GEN>
bool launch_third_wave(const IntegArgs<R>& a, int64_t n_groups, hipStream_t st) {
  if constexpr (sizeof(R) == 4 && NG == 16 && L > 1) {
    constexpr int64_t kSimds = 1024;
    const int64_t waves = n_groups * WPB;
    if (waves > 2 * kSimds && waves <= 3 * kSimds) {
      hipLaunchKernelGGL((k_rk4_group_lean<R, NG, PM, L, WPB, GEN>), dim3((unsigned)n_groups), dim3(64 * WPB),
                         0, st, a);
      return true;
    }
  }
  return false;
}

// The same for general Ito processes (IntegArgs::sde), instantiated in their
// own translation units.
template <typename R, int NG, int PM, int L, int WPB>
__global__ void __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(FMC_GROUP_MIN_WAVES)))
k_rk4_group_gen(IntegArgs<R> a) {
  constexpr int D = WPB == 1 ? 4 : 8;
  using Sh = GroupShape<R, NG, PM, L, WPB, D>;
  __shared__ __attribute__((aligned(16))) unsigned char lds[Sh::lds_bytes];
  GroupStats st{reinterpret_cast<double2*>(a.partial) + (int64_t)blockIdx.x * (a.S + 1) * a.V, 0};
  group_run<R, NG, PM, L, WPB, D, true>(a, blockIdx.x, lds, st, true);
}

}  // namespace fmc
