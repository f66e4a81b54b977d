// Scalar updates of the iteration states (finalize), shared by the finalize
// launch and by the passes that carry one as an extra block.
#pragma once
#include "fft_device.h"
#include "ffth_types.h"

namespace ffth {

__device__ static void fin_check(SolverState* st) {
  const double r = st->res;
  if (!(r == r) || r > 1e6) {
    st->flag = FLAG_DIVERGED;
    st->active = 0;
  } else if (r < st->tol) {
    st->flag = FLAG_CONVERGED;
    st->active = 0;
  } else if (st->iters >= st->max_iter) {
    st->active = 0;  // flag stays RUNNING: not converged
  }
}

// Partial sums are slot-major: part[k * nblk + block].  Each op names how
// many slots of each array it reads.
__device__ static void fin_slots(int op, int& nf, int& ni) {
  nf = 0;
  ni = 0;
  switch (op) {
    case FIN_LS_FIRST: nf = 1; ni = 1; break;
    case FIN_BS: ni = 1; break;
    case FIN_RESID_INIT: ni = 2; break;
    case FIN_CG_ALPHA: nf = 1; break;
    case FIN_CG_BETA: ni = 2; break;
    case FIN_OUTER: case FIN_OUTER_P: nf = 1; ni = 2; break;
    case FIN_PROJ: ni = 2; break;
    case FIN_CG3_INIT: nf = 3; break;
    case FIN_CG3: ni = 3; break;
    case FIN_BI_INIT: ni = 1; break;
    case FIN_BI_ALPHA: ni = 1; break;
    case FIN_BI_OMEGA: ni = 5; break;
    case FIN_SUMS_I: case FIN_O1RHS: ni = NRED; break;
  }
}

// Reduction asked of the FP32 inner solve that starts now.  The outer residual
// must still drop by need = 0.8 tol / res (the margin covers the FP32
// round-off of the correction); with at most tmin per solve that takes
// k = ceil(log need / log tmin) more solves, and the reduction is split evenly
// over them: every solve asks for need^(1/k) >= tmin.  Fewer restarts of the
// Krylov iteration than a fixed tmin, and no solve tighter than the sweeps
// still ahead require.
__device__ static double inner_target(double tmin, double outer_tol, double outer_res) {
  if (!(outer_res > 0.0) || !(tmin > 0.0) || !(tmin < 1.0)) return tmin;
  const double need = 0.8 * outer_tol / outer_res;
  if (!(need < 1.0)) return fmax(tmin, 0.5);
  if (need >= tmin) return need;
  const double k = ceil(log(need) / log(tmin));
  return fmax(tmin, pow(need, 1.0 / k));
}

// This thread's share (i = threadIdx.x mod NTF) of n partials, in a fixed
// order, with 8 independent accumulators so that 8 loads are in flight.
template <int NTF> __device__ __forceinline__ double strided_sum(const double* __restrict__ p, int n) {
  double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int i = threadIdx.x;
  for (; i + 7 * NTF < n; i += 8 * NTF) {
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] += p[i + u * NTF];
  }
  for (int u = 0; i < n; i += NTF, ++u) a[u & 7] += p[i];
  return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
}

// The gating flag of a load.  A pass that carries a finalize reads it in every
// block while the finalize's block may clear it, so both sides are atomic.
__device__ __forceinline__ bool flag_read(const SolverState* st) {
  return __hip_atomic_load(&st->active, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
__device__ __forceinline__ void flag_clear(SolverState* st) {
  __hip_atomic_store(&st->active, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Scalars of one iteration (the ops a pass may carry).
__device__ static void fin_iter(int op, SolverState* st, const double* sf, const double* si) {
  switch (op) {
    case FIN_CG_ALPHA: {
      const double pq = sf[0];
      if (!(pq > 0.0) || !(st->rr == st->rr)) {
        st->flag = FLAG_DIVERGED;
        flag_clear(st);
      } else {
        st->alpha = st->rr / pq;
      }
      break;
    }
    case FIN_CG3_INIT: {
      // three-term CG: rho_0 = <r,r>_C0, mu_0 = <r,Ar>_C0, gamma_0 = rho_0 / mu_0, omega_0 = 1
      if (!(sf[1] > 0.0) || !(sf[0] > 0.0)) {
        st->flag = sf[0] > 0.0 ? FLAG_DIVERGED : FLAG_CONVERGED;
        flag_clear(st);
        break;
      }
      st->rr = sf[0];
      st->alpha = sf[0] / sf[1];
      st->beta = 1.0;
      st->alpha_prev = 0.0;
      st->beta_prev = 1.0;
      st->xpend = 0;
      st->best_res = 1.0;
      st->best_it = 0;
      st->stalled = 0;
      st->first = 1;
      break;
    }
    case FIN_CG3: {
      // si = (rho_{k+1}, mu_{k+1}, ||r_{k+1}||^2); state holds rho_k, gamma_k, omega_k
      st->res = sqrt(si[2] / st->nb2);
      st->iters++;
      st->total++;
      const double g = si[0] / si[1];
      const double den = 1.0 - (g / st->alpha) * (si[0] / st->rr) / st->beta;
      const double om = 1.0 / den;
      st->first = 0;
      // stop before the scalars advance: a solve that stops keeps gamma_k,
      // omega_k (and gamma_{k-1}, omega_{k-1}) of its last iteration k, from
      // which k_cg3_finish forms x_{k+1} when k was even
      if (st->res < st->tol) {
        st->flag = FLAG_CONVERGED;
        flag_clear(st);
      } else if (!(si[1] > 0.0) || !(om == om) || !(fabs(om) < 1e6) || !(st->res == st->res) || st->res > 1e6) {
        st->flag = FLAG_DIVERGED;
        flag_clear(st);
      } else if (st->total >= st->max_iter) {
        // iteration budget (over all solves sharing the state: the mixed
        // scheme's inner solves count together) spent; flag stays RUNNING
        flag_clear(st);
      } else if (st->iters - st->best_it >= CG3_STALL && !(st->res < st->best_res)) {
        // no new smallest residual for CG3_STALL iterations: the rounding
        // floor of this precision; flag stays RUNNING
        st->stalled = 1;
        flag_clear(st);
      } else {
        st->rr = si[0];
        st->alpha_prev = st->alpha;
        st->beta_prev = st->beta;
        st->alpha = g;
        st->beta = om;
      }
      if (st->res < st->best_res) {
        st->best_res = st->res;
        st->best_it = st->iters;
      }
      // x is formed on odd iterations: after an even last one (iters odd) it is owed
      if (!flag_read(st)) st->xpend = st->iters & 1;
      break;
    }
  }
}

// Every other op: start of a solve, sweeps of the defect correction, sums.
__device__ static void fin_rest(int op, const Desc& d, SolverState* st, const double* sf, const double* si) {
  const double amu = fabs(d.mu0);
  switch (op) {
    case FIN_LS_FIRST: {
      st->nb2 = si[0];
      const double gs = st->gscale > 0.0 ? st->gscale : sqrt(sf[0]) / (2.0 * amu);
      st->iters = 0;
      st->first = 1;
      st->res = 1.0;
      if (sqrt(si[0]) <= st->guard_eps * gs) {
        st->flag = FLAG_ZERO_RHS;
        st->res = 0.0;
        st->active = 0;
      }
      break;
    }
    case FIN_BS:
      st->res = sqrt(si[0] / st->nb2);
      st->iters++;
      st->total++;
      fin_check(st);
      break;
    case FIN_RESID_INIT:
      st->rr = si[1];
      st->res = sqrt(si[0] / st->nb2);
      st->first = 1;
      if (st->res < st->tol) {
        st->flag = FLAG_CONVERGED;
        st->active = 0;
      }
      break;
    case FIN_CG_BETA:
      st->res = sqrt(si[1] / st->nb2);
      st->iters++;
      st->total++;
      st->beta = si[0] / st->rr;
      st->rr = si[0];
      st->first = 0;
      fin_check(st);
      break;
    case FIN_BI_INIT:
      // BiCGSTAB start: r_0 = b - A b, rho = <r^, r_0> = ||r_0||^2
      st->rr = si[0];
      st->res = sqrt(si[0] / st->nb2);
      st->alpha = st->omega = 1.0;
      st->beta = 0.0;
      st->first = 1;
      st->pending = 0;
      if (st->res < st->tol) {
        st->flag = FLAG_CONVERGED;
        st->active = 0;
      }
      break;
    case FIN_BI_ALPHA: {
      // alpha = rho / <r^, v>; the previous x update is applied by now
      st->pending = 0;
      const double rv = si[0];
      if (!(fabs(rv) > 0.0) || !(rv == rv)) {
        st->flag = FLAG_DIVERGED;
        st->active = 0;
      } else {
        st->alpha = st->rr / rv;
      }
      break;
    }
    case FIN_BI_OMEGA: {
      // si = (<t,s>, <t,t>, <r^,s>, <r^,t>, <s,s>)
      const double ts = si[0], tt = si[1];
      const double om = tt > 0.0 ? ts / tt : 0.0;
      const double rho = si[2] - om * si[3];
      const double r2 = fmax(0.0, si[4] - 2.0 * om * ts + om * om * tt);   // ||s - omega t||^2
      st->omega = om;
      st->pending = 1;
      st->first = 0;
      st->iters++;
      st->total++;
      st->res = sqrt(r2 / st->nb2);
      if (st->res < st->tol) {
        st->flag = FLAG_CONVERGED;
        st->active = 0;
      } else if (!(om != 0.0) || !(rho == rho) || !(fabs(rho) > 0.0)) {
        st->flag = FLAG_DIVERGED;   // breakdown
        st->active = 0;
      } else {
        st->beta = (rho / st->rr) * (st->alpha / om);
        st->rr = rho;
        fin_check(st);
      }
      break;
    }
    case FIN_PROJ: {
      // compatible part of the FP64 residual: restart the FP32 inner solve on it
      SolverState* in = d.st2;
      st->proj++;
      in->tol = inner_target(in->tol0, st->tol, st->res);
      in->active = si[0] > 0.0 ? 1 : 0;
      in->nb2 = si[0];
      in->dscale = si[0] > 0.0 ? sqrt(si[0] * d.inv_nvox) : 1.0;
      in->idscale = 1.0 / in->dscale;
      in->rr = si[1];
      in->first = 1;
      in->iters = 0;
      in->xpend = 0;
      in->flag = FLAG_RUNNING;
      in->res = 1.0;
      break;
    }
    case FIN_OUTER:
    case FIN_OUTER_P: {
      SolverState* in = d.st2;
      if (st->iters == 0) {
        st->nb2 = si[0];
        const double gs = st->gscale > 0.0 ? st->gscale : sqrt(sf[0]) / (2.0 * amu);
        if (sqrt(si[0]) <= st->guard_eps * gs) {
          st->flag = FLAG_ZERO_RHS;
          st->res = 0.0;
          st->active = 0;
          in->active = 0;
          break;
        }
      }
      st->res = sqrt(si[0] / st->nb2);
      st->iters++;
      st->fp64_apps++;
      if (!(st->res == st->res) || st->res > 1e6) {
        st->flag = FLAG_DIVERGED;
        st->active = 0;
      } else if (st->res < st->tol) {
        st->flag = FLAG_CONVERGED;
        st->active = 0;
      } else if (st->iters >= st->max_iter) {
        st->active = 0;
      }
      if (!st->active) {
        in->active = 0;
        in->xpend = 0;
      } else if (op == FIN_OUTER_P) {
        in->active = 0;  // the projection pass sets the inner solve up
      } else {
        in->active = 1;
        in->tol = inner_target(in->tol0, st->tol, st->res);
        in->nb2 = si[0];
        in->dscale = si[0] > 0.0 ? sqrt(si[0] * d.inv_nvox) : 1.0;
        in->idscale = 1.0 / in->dscale;
        in->rr = si[1];
        in->first = 1;
        in->iters = 0;
        in->xpend = 0;
        in->flag = FLAG_RUNNING;
        in->res = 1.0;
      }
      break;
    }
    case FIN_SUMS_I:
      for (int k = 0; k < NRED; ++k) st->sums[k] = si[k];
      break;
    case FIN_O1RHS:
      for (int k = 0; k < NRED; ++k) st->sums[k] = si[k];
      st->gscale = (sqrt(si[0]) + sqrt(si[1])) / (2.0 * amu);
      break;
  }
}

// Sums of the block partials of one batch entry and its scalar update, by a
// block of NTB threads, the first NTF of which sum (the others only meet its
// barriers).  Only the slots the op reads are summed, four at a time (red:
// NTF / 64 x 4 doubles of LDS).  ITER: only the ops of fin_iter.  The block is
// the only writer of the state while it runs.
template <int NTF, bool ITER, int NTB = NTF>
__device__ __forceinline__ void finalize_entry(const Desc& d, int op, int nblk_f, int nblk_i) {
  constexpr int NW = NTF / 64;
  __shared__ double red[NW][4];
  __shared__ double sums[2 * NRED];
  SolverState* st = d.st;
  if (!flag_read(st)) return;
  if (nblk_i < 0) nblk_i = d.nblk_multi;   // multi-size launch: each entry's own block count
  int nf, ni;
  fin_slots(op, nf, ni);
  const int ns = nf + ni, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int k0 = 0; k0 < ns; k0 += 4) {
    if (NTB == NTF || w < NW) {
      double a[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + u, n = k < nf ? nblk_f : nblk_i;
        const double* p = k < nf ? d.part_f + (long)k * nblk_f : d.part_i + (long)(k - nf) * nblk_i;
        a[u] = k < ns ? strided_sum<NTF>(p, n) : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (k0 + u < ns) a[u] = wave_sum(a[u]);
        if (lane == 0) red[w][u] = a[u];
      }
    }
    __syncthreads();
    if (threadIdx.x < 4 && k0 + (int)threadIdx.x < ns) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < NW; ++i) s += red[i][threadIdx.x];
      const int k = k0 + threadIdx.x;
      sums[k < nf ? k : NRED + k - nf] = s;
    }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  if (op == FIN_CG_ALPHA || op == FIN_CG3_INIT || op == FIN_CG3) fin_iter(op, st, sums, sums + NRED);
  else if constexpr (!ITER) fin_rest(op, d, st, sums, sums + NRED);
}

}  // namespace ffth
