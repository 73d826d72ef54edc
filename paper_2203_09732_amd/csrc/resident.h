// MINRES with every vector of one realization on chip: the recurrence vectors
// in registers (a thread owns the same rows for the whole solve), the vector
// the product gathers from in LDS, and the neighbour of every (row, bond) as
// a 16-bit LDS offset in registers, so that an iteration touches no memory
// beyond the compute unit.
//
// The recurrences of Alg. 2 are run on u = M^{1/2} q = M^{-1/2} z, i.e. the
// same Lanczos process written for M^{-1/2} A M^{-1/2} (rs = M^{-1/2}):
//   u_{k+1} = (rs p_k) / beta_k - (alpha_k / beta_k) u_k - (beta_k / beta_{k-1}) u_{k-1},
// p_k = A q_k, q_k = rs u_k, beta_k^2 = u_k . u_k = q_k . z_k, and the search
// directions and x likewise (x = rs x~). One vector takes the place of z and
// q, and no division is left in the loop.
#pragma once

#include "rows.h"

namespace mbl {

// Scalars of an iteration shared by the workgroup: for iteration k, 1 / beta_k
// and beta_k / beta_{k-1}; for the d/x update of iteration k - 1, its
// coefficients; whether the solve is done after iteration k - 1.
struct ResidentCoef {
  double ib, c3;
  double ibp, de, ep, ig, tau;
  int done;
};

// 1 / sqrt(v): the hardware estimate and two Newton steps (to about an ulp; 0,
// infinities and NaN as the estimate gives them). A square root and a division
// one after the other take three times as long, on the critical path.
__device__ __forceinline__ double rsqrt_newton(double v) {
  const double y0 = __builtin_amdgcn_rsq(v);
  double y = y0;
  y = fma(0.5 * y, fma(-(v * y), y, 1.0), y);
  y = fma(0.5 * y, fma(-(v * y), y, 1.0), y);
  return v > 0.0 && v < INFINITY ? y : y0;
}

// The scalar recurrence of Alg. 2, kept by one wave.
struct ResidentScalars {
  double beta = 1.0, ib = 0.0, ib_old = 0.0, qz_ = 0.0;   // beta_k, 1 / beta_k, 1 / beta_{k-1}
  double c = 1.0, s = 0.0, dhat = 0.0, eps = 0.0, phi = 0.0;
  double delta = 0.0, gamma_hat = 0.0;  // of iteration k - 1, from its alpha
  bool bad = false;
  // after iteration k - 1's alpha is known
  __device__ __forceinline__ void rotate(double alpha) {
    delta = c * dhat + s * alpha;
    gamma_hat = -s * dhat + c * alpha;
    bad = bad || !isfinite(alpha);
  }
  // Before iteration k: beta_k from qz = u_k . u_k. Fills co.ib and co.c3.
  __device__ __forceinline__ void lanczos(int64_t k, double qz, ResidentCoef& co) {
    ib_old = ib;
    ib = rsqrt_newton(qz);
    const double b0 = qz * ib;   // the root, with one correction (half an ulp)
    beta = qz == 0.0 ? 0.0 : fma(0.5 * ib, fma(-b0, b0, qz), b0);
    qz_ = qz;
    co.ib = ib;
    co.c3 = beta * (k == 1 ? 1.0 : ib_old);
  }
  // then the Givens step of iteration k - 1 (k >= 2): the rest of co
  __device__ __forceinline__ void givens(int64_t k, double tol, int64_t kmax, ResidentCoef& co) {
    co.ibp = ib_old;
    if (k == 1) {
      phi = beta;
      bad = !isfinite(beta);
      co.de = co.ep = co.ig = co.tau = 0.0;
    } else {
      const double ig = rsqrt_newton(gamma_hat * gamma_hat + qz_);
      co.de = delta;
      co.ep = eps;
      co.ig = ig;
      eps = s * beta;
      dhat = c * beta;
      c = gamma_hat * ig;
      s = beta * ig;
      co.tau = c * phi;
      phi = -s * phi;
      bad = bad || !isfinite(phi) || !isfinite(beta);
    }
    co.done = (bad || !(fabs(phi) >= tol && k - 1 < kmax)) ? 1 : 0;
  }
};

// One workgroup, one realization, n < RPT * NT. The caller fills, for the
// thread's rows tid + i NT (i < RPT): nb[i][b] = two byte offsets into q of
// the neighbours on bonds 2b and 2b + 1 (8 n, a place that stays 0, for a bond
// that is not antiparallel), the diagonal dg[i] (shift included), rs[i], and
// u[i] = rs b with b the right-hand side; rows from n on have u = rs = dg = 0
// and only offsets 8 n, so they stay 0. On return x[i] = rs x~ is the
// solution, from x0 = 0. q: RPT * NT doubles of LDS; red: 2 * waves doubles.
//
// What bounds it: the LDS gathers (L 8-byte reads per row and iteration, at
// about 6 cycles a wave instruction), then two workgroup reductions.
//
// DEFL: the operator is A + theta v v^T (v per row; red: 3 * waves doubles).
template <int NPAIR, int RPT, int NT, bool DEFL = false>
__device__ __forceinline__ void resident_minres(
    const uint32_t (&nb)[RPT][NPAIR], const double (&dg)[RPT],
    const double (&rs)[RPT], double (&u)[RPT], double (&x)[RPT], double* q, double* red, ResidentCoef* co,
    double tol, int64_t kmax, int64_t& iters, double& phi_out, bool& bad_out,
    const double (&v)[DEFL ? RPT : 1], double theta) {
  constexpr int NW = NT / 64;
  constexpr int SW = NW - 1;   // the wave that keeps the scalars (it owns the fewest rows)
  const int lane = threadIdx.x & 63;
  const int wave = (int)uni(threadIdx.x >> 6);
  double* const qw = q + threadIdx.x;   // this thread's rows
  double* red1 = red;
  double* red2 = red + NW;
  double* red3 = red + 2 * NW;
  double up[RPT], d1[RPT], d0[RPT];
  double acc = 0.0, accv = 0.0;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    up[i] = d1[i] = d0[i] = x[i] = 0.0;
    acc += u[i] * u[i];
    if (DEFL) accv += v[i] * (u[i] * rs[i]);
    qw[i * NT] = u[i] * rs[i];
  }
  auto put = [&](double v, double* r) {
    v = wave_sum(v);
    if (lane == 0) r[wave] = v;
  };
  auto total = [&](const double* r) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += r[w];
    return t;
  };
  put(acc, red2);
  if (DEFL) put(accv, red3);
  __syncthreads();
  ResidentScalars sc;
  double alpha = 0.0;
  int64_t k = 0;
  // iteration k on (u_k, u_{k-1}, d_{k-2}, d_{k-3}); u_{k-1} is overwritten by
  // u_{k+1} and d_{k-3} by d_{k-1}. Returns false when the solve was done
  // after iteration k - 1 (then only its d/x update has been taken).
  auto iteration = [&](double (&uk)[RPT], double (&um)[RPT], double (&da)[RPT],
                       double (&db)[RPT]) -> bool {
    ++k;
    if (wave == SW) {
      ResidentCoef c;
      if (k > 1) sc.rotate(alpha);
      sc.lanczos(k, total(red2), c);
      sc.givens(k, tol, kmax, c);
      if (lane == 0) *co = c;
    }
    const double tv = DEFL ? theta * total(red3) : 0.0;
    double p[RPT];
    double a1 = 0.0;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      double off = 0.0;
#pragma unroll
      for (int b = 0; b < NPAIR; ++b) {
        uint32_t w = nb[i][b];
        asm volatile("" : "+v"(w));   // keep the pair packed: unpacked in the loop, not before it
        off += *reinterpret_cast<const double*>(reinterpret_cast<const char*>(q) + (w & 0xffffu));
        off += *reinterpret_cast<const double*>(reinterpret_cast<const char*>(q) + (w >> 16));
      }
      const double qi = uk[i] * rs[i];
      p[i] = dg[i] * qi + 0.5 * off;
      if (DEFL) p[i] += tv * v[i];
      a1 += qi * p[i];
    }
    put(a1, red1);
    __syncthreads();
    const ResidentCoef c = *co;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const double d = (um[i] * c.ibp - c.de * da[i] - c.ep * db[i]) * c.ig;
      db[i] = d;
      x[i] += c.tau * d;
    }
    if (c.done) return false;
    const double qp = total(red1);
    const double c2 = qp * c.ib * c.ib * c.ib;
    alpha = qp * c.ib * c.ib;
    double a2 = 0.0, av = 0.0;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const double un = c.ib * (p[i] * rs[i]) - c2 * uk[i] - c.c3 * um[i];
      um[i] = un;
      a2 += un * un;
      if (DEFL) av += v[i] * (un * rs[i]);
      qw[i * NT] = un * rs[i];
    }
    put(a2, red2);
    if (DEFL) put(av, red3);
    __syncthreads();
    return true;
  };
  for (;;) {
    if (!iteration(u, up, d1, d0)) break;
    if (!iteration(up, u, d0, d1)) break;
  }
#pragma unroll
  for (int i = 0; i < RPT; ++i) x[i] *= rs[i];
  // the scalars of the last step to every thread
  if (wave == SW && lane == 0) {
    red2[0] = sc.phi;
    red2[1] = sc.bad ? 1.0 : 0.0;
  }
  __syncthreads();
  phi_out = red2[0];
  bad_out = red2[1] != 0.0;
  iters = k - 1;
  __syncthreads();
}

}  // namespace mbl
