// Generic HIP kernels of the projection path, templated on the constraint model.
//
// Mapping: one configuration per lane; the lane's FP64 iterate lives in LDS (a column
// of a [D][blockDim] array, conflict-free); the kinematic constants are read with scalar
// loads (wave-uniform, so they occupy scalar registers), as are the boxes of the scene in the exact
// check; everything else is in registers. The hot
// loop (Alg. 2 ParallelProject with getDescentStep on one stacked block) per iteration:
//   1. residual pass, FP64: forward kinematics, F(q), ||F||^2, and the per-block data
//      the Jacobian columns need;
//   2. convergence test ||F||^2 < tol^2 (per lane; a wave leaves the loop when every
//      lane is done);
//   3. Gram pass in the step precision: the tree is walked again, each Jacobian column
//      is formed and folded into J J^T (structural nonzeros only); J is never stored;
//   4. in-register Cholesky of J J^T (+ lambda I) with the condition estimate
//      (max L_ii / min L_ii)^2 and forward/back substitution for y = (J J^T)^-1 F;
//      lanes whose estimate exceeds the threshold, or whose factorisation fails,
//      redo 1, 3 and 4 in FP64;
//   5. J^T y pass (a third walk), dq = alpha J^T y, optional
//      divergence exit, q <- q - dq.
// Passes 1, 3 and 5 are those of StepOf<Model>: the model's own, or the leaf-to-root walks.
// The persistent variant refills a lane from a device work queue as soon as its
// configuration finishes, so lanes do not idle until the slowest configuration of
// their wave converges.
#pragma once

#include "common.hpp"
#include "trig.hpp"

namespace mc {

struct ProjArgs {
  const DevProblem* P;
  int64_t n;          // configurations handled by this launch
  int64_t base;       // index of the first one in the caller's arrays
  const void* q_in;
  int64_t ld_in;
  void* q_out;
  int64_t ld_out;
  int8_t* status;
  int8_t* iters;
  void* resid;
  uint8_t* verdict;   // plain fused kernel only
  double tol2, alpha, lambda, max_step, cond_thr;
  int32_t max_iter;
  int32_t check;
  int32_t outer;          // 1: the outer form of the step, (J^T J + lambda I)^-1 J^T F (families with D <= kOuterMaxD)
  unsigned int* counter;  // persistent: queue head (0 at the launch)
  unsigned int* clear;    // persistent: the counters of the next call, zeroed here (nullptr: none)
  int64_t n_static;       // persistent: configurations [0, n_static) are taken by thread id
  // FP32 mode: configurations whose FP32 step fails (factorisation or condition estimate) are
  // handed to the FP64 tail kernel through this queue: defer_ik[2s], defer_ik[2s+1] = index and
  // steps taken, defer_q[c * defer_cap + s] = FP64 iterate.
  unsigned int* defer_count;
  int32_t* defer_ik;
  double* defer_q;
  int64_t defer_cap;
  // Fused collision check: converged configurations whose broad-phase test found a link near
  // the obstacles are queued here for the exact check
  // (index in chk_idx[s], FP64 configuration at chk_q[c * defer_cap + s]).
  unsigned int* chk_count;
  int32_t* chk_idx;
  double* chk_q;
  int32_t n_sph, n_obs;   // robot and obstacle spheres (LDS size of the exact-check kernel)
  int32_t chk_lanes;      // exact check: lanes per queued configuration (0: chk_long; 1, 2, 4, 8, 16, 64)
  int32_t chk_long;       // exact check: lanes per configuration as tuned or by the scene, with chk_lanes = 0 (2, 4, 8 or 16
                          // on long queues and 64 on short ones; 0 or 1: one lane per configuration on every queue)
};

constexpr int ST_DEFER = -2;  // internal: continue this configuration with FP64 steps
constexpr int kCounters = 4;   // queue counters of a call

template <class IO>
__device__ __forceinline__ double ld_io(const void* p, int64_t k) { return double(static_cast<const IO*>(p)[k]); }
template <class IO>
__device__ __forceinline__ void st_io(void* p, int64_t k, double v) { static_cast<IO*>(p)[k] = IO(v); }

template <class IO>
struct QGlob {  // configuration i of a [D][ld] array in global memory
  const IO* p;
  int64_t ld, i;
  int dof;
  __device__ __forceinline__ double at(int j) const { return j < dof ? double(p[j * ld + i]) : 0.0; }
  template <class U>
  __device__ __forceinline__ double at(int j, U) const { return at(j); }
  __device__ __forceinline__ double get(int j) const { return at(j); }
  __device__ __forceinline__ QGlob fresh() const { return *this; }
};

// ------------------------------------------------------------------ Cholesky
// Rows a lane has dropped (bits of Model::DROPPABLE; none for models that never drop rows).
template <class Model, class SDT>
__device__ __forceinline__ uint32_t drop_bits(const SDT& sd) {
  if constexpr (Model::DROPPABLE != 0) return sd.drop;
  else return 0u;
}

// In-place right-looking Cholesky of the packed lower triangle G (structural zeros of the
// factor skipped at compile time). Returns false on a non-positive or non-finite pivot, or a
// pivot below floor. invd receives 1 / L_ii; kappa the estimate (max L_ii / min L_ii)^2.
// A dropped row (its G row and column are zero) gets the unit pivot and takes no part in kappa.
template <class Model, class S, uint32_t RM = ~uint32_t(0)>
__device__ __forceinline__ bool cholesky(S* G, S* invd, S& kappa, S floor, uint32_t drop = 0u) {
  constexpr int M = Model::M;
  bool ok = true;
  S dmin = S(3.0e38), dmax = S(0);
  sfor<0, M>([&](auto K) {
    constexpr int k = decltype(K)::value;
    if constexpr (((RM >> k) & 1u) != 0) {
    bool dk = false;
    if constexpr (((Model::DROPPABLE >> k) & 1u) != 0) dk = ((drop >> k) & 1u) != 0;
    const S d = dk ? S(1) : G[pidx(k, k)];
    ok = ok && (dk || ((d > floor) && finite_t(d)));
    const S r = rsqrt_t(d);
    const S l = d * r;
    G[pidx(k, k)] = l;
    invd[k] = r;
    dmin = (dk || !(l < dmin)) ? dmin : l;
    dmax = (dk || !(l > dmax)) ? dmax : l;
    sfor<k + 1, M>([&](auto I) {
      constexpr int i = decltype(I)::value;
      if constexpr (Model::lnz(i, k) && ((RM >> i) & 1u)) G[pidx(i, k)] *= r;
    });
    sfor<k + 1, M>([&](auto I) {
      constexpr int i = decltype(I)::value;
      if constexpr (Model::lnz(i, k) && ((RM >> i) & 1u)) {
        sfor<k + 1, i + 1>([&](auto Jx) {
          constexpr int j = decltype(Jx)::value;
          if constexpr (Model::lnz(j, k) && ((RM >> j) & 1u)) G[pidx(i, j)] -= G[pidx(i, k)] * G[pidx(j, k)];
        });
      }
    });
    }
  });
  S ratio = dmax / dmin;
  if constexpr (Model::DROPPABLE != 0) ratio = dmax > S(0) ? ratio : S(0);  // every row dropped
  kappa = ratio * ratio;
  return ok && finite_t(kappa);
}

// Solve L L^T y = b in place (b overwritten by y).
template <class Model, class S, uint32_t RM = ~uint32_t(0)>
__device__ __forceinline__ void chol_solve(const S* L, const S* invd, S* y) {
  constexpr int M = Model::M;
  sfor<0, M>([&](auto I) {
    constexpr int i = decltype(I)::value;
    if constexpr ((RM >> i) & 1u) {
      S acc = y[i];
      sfor<0, i>([&](auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (Model::lnz(i, k) && ((RM >> k) & 1u)) acc -= L[pidx(i, k)] * y[k];
      });
      y[i] = acc * invd[i];
    }
  });
  sfor<0, M>([&](auto I) {
    constexpr int i = M - 1 - decltype(I)::value;
    if constexpr ((RM >> i) & 1u) {
      S acc = y[i];
      sfor<i + 1, M>([&](auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (Model::lnz(k, i) && ((RM >> k) & 1u)) acc -= L[pidx(k, i)] * y[k];
      });
      y[i] = acc * invd[i];
    }
  });
}

constexpr float kFloorF32 = 0.0f;
constexpr double kFloorF64 = 1e-24;  // pivot floor relative to the largest Gram diagonal entry

// One descent step in precision S: dq = J^T (J J^T + lambda I)^-1 rhs (rhs = F for Newton;
// overwritten). Returns false when the factorisation fails or, in FP32, its condition estimate
// exceeds the call's threshold.
// RM restricts the system to the rows of one block (cyclic mode).
template <class Model, class S, uint32_t RM = ~uint32_t(0), class Q, class TR, class SDT>
__device__ __forceinline__ bool descent_step(const Q& q, S* rhs, const SDT& sd, const TR& tr, const Consts& C, S floor_rel,
                                             S* dq) {
  constexpr int M = Model::M;
  using W = typename StepOf<Model>::type;
  S G[M * (M + 1) / 2];
  W::template gram<S, RM>(q, C, sd, tr, G);
  const ProjArgs& a = kernarg<ProjArgs>();
  if (a.lambda > 0.0) W::template add_lambda<S, RM>(G, rhs, S(a.lambda), tr);
  S maxd = S(0);
  sfor<0, M>([&](auto I) {
    constexpr int i = decltype(I)::value;
    if constexpr ((RM >> i) & 1u) maxd = G[pidx(i, i)] > maxd ? G[pidx(i, i)] : maxd;
  });
  S invd[M], kappa;
  if (!cholesky<Model, S, RM>(G, invd, kappa, floor_rel * maxd, drop_bits<Model>(sd))) return false;
  if constexpr (std::is_same<S, float>::value)
    if (!(double(kappa) <= kernarg<ProjArgs>().cond_thr)) return false;
  chol_solve<Model, S, RM>(G, invd, rhs);
  W::template jty<S, RM>(q, C, sd, tr, rhs, dq);
  return true;
}

// ------------------------------------------------------------------ outer form of the step
// The step's alternative form (Alg. 2 getDescentStep; Sec. IV-A provides the inner and the outer
// pseudo-inverse): dq = (J^T J + lambda I)^-1 J^T F, a d x d system, for lambda > 0. Built for the
// families with d <= kOuterMaxD, whose dense J and packed d x d factor fit a lane's registers.
constexpr int kOuterMaxD = 16;

// Dense packed-lower Cholesky of an N x N matrix in place (all entries), with the same conventions
// as cholesky(): false on a pivot <= floor or non-finite; invd = 1 / L_ii; kappa = (max / min L_ii)^2.
template <int N, class S>
__device__ __forceinline__ bool dense_cholesky(S* A, S* invd, S& kappa, S floor) {
  bool ok = true;
  S dmin = S(3.0e38), dmax = S(0);
  sfor<0, N>([&](auto K) {
    constexpr int k = decltype(K)::value;
    const S d = A[pidx(k, k)];
    ok = ok && (d > floor) && finite_t(d);
    const S r = rsqrt_t(d);
    const S l = d * r;
    A[pidx(k, k)] = l;
    invd[k] = r;
    dmin = l < dmin ? l : dmin;
    dmax = l > dmax ? l : dmax;
    sfor<k + 1, N>([&](auto I) { A[pidx(decltype(I)::value, k)] *= r; });
    sfor<k + 1, N>([&](auto I) {
      constexpr int i = decltype(I)::value;
      sfor<k + 1, i + 1>([&](auto Jx) {
        constexpr int j = decltype(Jx)::value;
        A[pidx(i, j)] -= A[pidx(i, k)] * A[pidx(j, k)];
      });
    });
  });
  const S ratio = dmax / dmin;
  kappa = ratio * ratio;
  return ok && finite_t(kappa);
}

template <int N, class S>
__device__ __forceinline__ void dense_solve(const S* L, const S* invd, S* y) {
  sfor<0, N>([&](auto I) {
    constexpr int i = decltype(I)::value;
    S acc = y[i];
    sfor<0, i>([&](auto K) { acc -= L[pidx(i, decltype(K)::value)] * y[decltype(K)::value]; });
    y[i] = acc * invd[i];
  });
  sfor<0, N>([&](auto I) {
    constexpr int i = N - 1 - decltype(I)::value;
    S acc = y[i];
    sfor<i + 1, N>([&](auto K) { acc -= L[pidx(decltype(K)::value, i)] * y[decltype(K)::value]; });
    y[i] = acc * invd[i];
  });
}

// dq = (J^T J + lambda I)^-1 J^T rhs with the dense Jacobian of the step pass (dropped rows are zero
// rows of J and need no special case: lambda > 0 keeps the d x d matrix positive definite).
template <class Model, class S, class Q>
__device__ __forceinline__ bool descent_step_outer(const Q& q, const S* rhs, const typename Model::template SD<S>& sd,
                                                   const Consts& C, double lambda, double cond_thr, S floor_rel, S* dq) {
  constexpr int D = Model::D, M = Model::M;
  S J[M * D];
  Model::template jacobian<S>(q, C, sd, J);
  S A[D * (D + 1) / 2];
  S maxd = S(0);
  sfor<0, D>([&](auto I) {
    constexpr int i = decltype(I)::value;
    sfor<0, i + 1>([&](auto K) {
      constexpr int k = decltype(K)::value;
      S acc = (i == k) ? S(lambda) : S(0);
      for (int r = 0; r < M; ++r) acc += J[r * D + i] * J[r * D + k];
      A[pidx(i, k)] = acc;
    });
    maxd = A[pidx(i, i)] > maxd ? A[pidx(i, i)] : maxd;
    S b = S(0);
    for (int r = 0; r < M; ++r) b += J[r * D + i] * rhs[r];
    dq[i] = b;
  });
  S invd[D], kappa;
  if (!dense_cholesky<D, S>(A, invd, kappa, floor_rel * maxd)) return false;
  if (!(double(kappa) <= cond_thr)) return false;
  dense_solve<D, S>(A, invd, dq);
  return true;
}

// Apply dq (scaled by alpha) with the divergence test. Returns -1 after the update or a status.
template <class Model, class S>
__device__ __forceinline__ int apply_step(const QLds& q, const S* dq) {
  constexpr int D = Model::D;
  const ProjArgs& a = kernarg<ProjArgs>();
  const QLds qf = q.fresh();
  double x[D], s2 = 0.0;
  for (int j = 0; j < D; ++j) {
    x[j] = qf.get(j);
    const double d = a.alpha * double(dq[j]);
    s2 += d * d;
  }
  if (!finite_t(s2)) return ST_NONFINITE;
  if (a.max_step > 0.0 && s2 > a.max_step * a.max_step) return ST_DIVERGED;
  for (int j = 0; j < D; ++j) q.set(j, x[j] - a.alpha * double(dq[j]));
  return -1;
}

// One Newton iteration for one lane: residual and convergence test in FP64, then the step in
// precision S. Returns -1 after taking a step, else the final status; in FP32 mode ST_DEFER
// when the FP32 factorisation fails or its condition estimate exceeds the threshold (the
// iteration is then redone with an FP64 step, and the configuration stays in FP64 until it
// ends). OUTER: the outer form of the step, on the model's own rows.
template <class Model, class S, bool OUTER, class TR>
__device__ __forceinline__ int newton_iteration(const QLds& q, const TR& tr, int& k, const Consts& C, double& resid) {
  constexpr int D = Model::D, M = Model::M;
  using W = std::conditional_t<OUTER, Direct<Model>, typename StepOf<Model>::type>;
  constexpr bool f32 = std::is_same<S, float>::value;
  typename W::template SD<S> sd;
  S F[M];
  const double n2 = W::template residual<S>(q, C, F, sd, tr);
  const ProjArgs& a = kernarg<ProjArgs>();
  resid = sqrt(n2);
  if (!finite_t(n2)) return ST_NONFINITE;
  if (n2 < a.tol2) return ST_CONVERGED;
  if (k >= a.max_iter) return ST_MAX_ITER;
  S dq[D];
  const S floor_rel = f32 ? S(kFloorF32) : S(kFloorF64);
  bool ok;
  if constexpr (OUTER) ok = descent_step_outer<Model, S>(q, F, sd, C, a.lambda, f32 ? a.cond_thr : 1e300, floor_rel, dq);
  else ok = descent_step<Model, S>(q, F, sd, tr, C, floor_rel, dq);
  if (!ok) return f32 ? ST_DEFER : ST_SINGULAR;
  const int st = apply_step<Model, S>(q, dq);
  if (st < 0) ++k;
  return st;
}

// One iteration of the cyclic mode (Alg. 2, getDescentStep looping over the constraints, Sec.
// IV-C): the full residual and the convergence test, then one min-norm step per constraint block
// in order, each taken from the configuration the previous block left; the divergence test
// (MaxDistance) applies to the displacement of the whole iteration. q0 receives the iterate at
// the start of the iteration. In FP32 mode a failed factorisation in any block restores that
// iterate and returns ST_DEFER (the iteration is redone in FP64).
template <class Model, class S, class TR>
__device__ __forceinline__ int cyclic_iteration(const QLds& q, const QLds& q0, const TR& tr, int& k, const Consts& C,
                                                double& resid) {
  constexpr int D = Model::D, M = Model::M, NB = Model::NBLK;
  constexpr bool f32 = std::is_same<S, float>::value;
  using W = typename StepOf<Model>::type;
  typename W::template SD<S> sd;
  S F[M];
  const double n2 = W::template residual<S>(q, C, F, sd, tr);
  const ProjArgs& a = kernarg<ProjArgs>();
  resid = sqrt(n2);
  if (!finite_t(n2)) return ST_NONFINITE;
  if (n2 < a.tol2) return ST_CONVERGED;
  if (k >= a.max_iter) return ST_MAX_ITER;
  for (int c = 0; c < D; ++c) q0.set(c, q.at(c));
  int st = -1;
  bool failed = false;
  sfor<0, NB>([&](auto BI) {
    constexpr int b = decltype(BI)::value;
    constexpr uint32_t RM = Model::block_rows_mask(b);
    if (st < 0 && !failed) {
      // the first block steps from the iterate whose residual is already in F and sd
      if constexpr (b > 0) W::template residual<S, RM>(q, C, F, sd, tr);
      S dq[D];
      if (!descent_step<Model, S, RM>(q, F, sd, tr, C, f32 ? S(kFloorF32) : S(kFloorF64), dq)) {
        failed = true;
      } else {
        double s2 = 0.0;
        for (int j = 0; j < D; ++j) {
          const double dj = a.alpha * double(dq[j]);
          s2 += dj * dj;
        }
        if (!finite_t(s2)) st = ST_NONFINITE;
        else
          for (int j = 0; j < D; ++j) q.set(j, q.at(j) - a.alpha * double(dq[j]));
      }
    }
  });
  if (failed) {
    if constexpr (f32) {
      for (int c = 0; c < D; ++c) q.set(c, q0.at(c));
      return ST_DEFER;
    } else {
      return ST_SINGULAR;
    }
  }
  if (st >= 0) return st;
  if (a.max_step > 0.0) {
    double s2 = 0.0;
    for (int c = 0; c < D; ++c) {
      const double t = q.at(c) - q0.at(c);
      s2 += t * t;
    }
    if (s2 > a.max_step * a.max_step) {
      for (int c = 0; c < D; ++c) q.set(c, q0.at(c));
      return ST_DIVERGED;
    }
  }
  ++k;
  return -1;
}

// The step a kernel is built for.
enum : int { STACKED = 0, CYCLIC = 1, OUTER = 2 };

// One iteration of a build.
template <class Model, class S, int MODE, class TR>
__device__ __forceinline__ int iteration(const QLds& q, const QLds& q0, const TR& tr, int& k, const Consts& C, double& resid) {
  if constexpr (MODE == CYCLIC) return cyclic_iteration<Model, S>(q, q0, tr, k, C, resid);
  else return newton_iteration<Model, S, MODE == OUTER>(q, tr, k, C, resid);
}

// Run one configuration to the end with FP64 steps.
template <class Model, int MODE, class TR>
__device__ __forceinline__ int finish_fp64(const QLds& q, const QLds& q0, const TR& tr, int& k, const Consts& C, double& resid) {
  int st;
  do {
    st = iteration<Model, double, MODE>(q, q0, tr, k, C, resid);
  } while (st < 0);
  return st;
}

// LDS of the projection and VJP kernels, in doubles: the sine table of the models that use one, the
// per-wave [D][64] iterate tiles, what else the kernel keeps per lane, and last the tiles of sines and
// cosines (TILE; two floats per entry).
template <class Model>
constexpr int kTabDoubles = StepOf<Model>::type::trig ? kSinTabDoubles : 0;
template <class Model, bool TILE, bool EXACT = true>
using TrigFor = std::conditional_t<!StepOf<Model>::type::trig, TrigNone, std::conditional_t<TILE, TrigTile, TrigLiveOf<EXACT>>>;
// The lane's trig source; tile: the kernel's first double of trig tiles. The table is staged by the whole
// block, before any lane leaves.
template <class Model, bool TILE, bool EXACT = true>
__device__ __forceinline__ TrigFor<Model, TILE, EXACT> make_trig(double* smem, double* tile) {
  TrigFor<Model, TILE, EXACT> t;
  if constexpr (StepOf<Model>::type::trig) {
    stage_sin_tab(smem);
    __syncthreads();
    t.tab = (SinTabP)smem;
    if constexpr (TILE)
      t.base = (TrigTile::LP)(reinterpret_cast<TrigTile::V2*>(tile) + (int(threadIdx.x) >> 6) * (Model::D * 64) + (int(threadIdx.x) & 63));
  }
  return t;
}
// FP32 projections of the models with trig tiles keep one (the cyclic build has no LDS left for it).
template <class Model, class S, int MODE>
constexpr bool kTrigTile = StepOf<Model>::type::trig && std::is_same<S, float>::value && MODE == STACKED;
// Dynamic LDS of a projection kernel, in bytes.
template <class Model, int MODE, bool TILE>
constexpr size_t projection_lds(int block) {
  return 8 * (size_t(kTabDoubles<Model>) + size_t(Model::D) * size_t(block) * (1 + (MODE == CYCLIC ? 1 : 0) + (TILE ? 1 : 0)));
}

// Configuration dimension: a compile-time constant where the model fixes it (the per-coordinate
// guards of the load and store loops then fold away), else the scene's value.
template <class Model>
__device__ __forceinline__ int dof_of(const Consts& C) {
  if constexpr (Model::fixed_dof) return Model::D;
  else return C.dof;
}

// Column c of configuration i in a [D][ld] array sits at (c ld + i); the pointer is bumped by
// an opaque ld so the D addresses are formed one after another rather than all up front.
template <class Model, class IO>
__device__ __forceinline__ void load_q(const ProjArgs& a, int dof, int64_t i, const QLds& q) {
  const IO* p = static_cast<const IO*>(a.q_in) + a.base + i;
  const int64_t ld = a.ld_in;
  IO x[Model::D];  // every coordinate requested before the first is waited for
  for (int c = 0; c < Model::D; ++c) {
    x[c] = c < dof ? *p : IO(0);
    p += after(ld, c);
  }
  __builtin_amdgcn_sched_barrier(0);
  for (int c = 0; c < Model::D; ++c) q.set(c, double(x[c]));
}

template <class Model, class IO>
__device__ __forceinline__ void store_result(const ProjArgs& a, int dof, int64_t i, const QLds& q, int st, int k,
                                             double resid) {
  IO* p = static_cast<IO*>(a.q_out) + a.base + i;
  const int64_t ld = a.ld_out;
  const QLds qf = q.fresh();
  for (int c0 = 0; c0 < Model::D; c0 += 12) {  // twelve coordinates at a time
    double x[12];
    for (int c = 0; c < 12; ++c) x[c] = c0 + c < Model::D ? qf.get(c0 + c) : 0.0;
    __builtin_amdgcn_sched_barrier(0);
    for (int c = 0; c < 12; ++c) {
      if (c0 + c < dof && c0 + c < Model::D) *p = IO(x[c]);
      p += after(ld, c);
    }
  }
  a.status[a.base + i] = int8_t(st);
  a.iters[a.base + i] = int8_t(k);
  st_io<IO>(a.resid, a.base + i, resid);
}

// Append the calling lane's FP64 configuration to a queue (slot < defer_cap: the queues are
// sized for the batch).
template <class Model, class Q>
__device__ __forceinline__ unsigned queue_q(const Q& q, unsigned* count, double* qbuf, int64_t cap) {
  const unsigned slot = atomicAdd(count, 1u);
  double* dst = qbuf + slot;
  double x[Model::D];
  for (int c = 0; c < Model::D; ++c) x[c] = q.get(c);
  __builtin_amdgcn_sched_barrier(0);
  for (int c = 0; c < Model::D; ++c) {
    *dst = x[c];
    dst += after(cap, c);
  }
  return slot;
}

template <class Model, class IO, class Q>
__device__ __forceinline__ void load_queued(const double* qbuf, int64_t cap, int64_t slot, const Q& q) {
  const double* src = qbuf + slot;
  double x[Model::D];
  for (int c = 0; c < Model::D; ++c) {
    x[c] = *src;
    src += after(cap, c);
  }
  __builtin_amdgcn_sched_barrier(0);
  for (int c = 0; c < Model::D; ++c) q.set(c, x[c]);
}

// Collision verdict of a configuration that ended with status st (exact check in-line).
template <class Model>
__device__ __forceinline__ uint8_t verdict_inline(const QLds& q, const Consts& C, const ProjArgs& a, int st) {
  if (!a.check || st != ST_CONVERGED) return V_UNCHECKED;
  const CollConsts& K = coll_of(a.P);
  return Model::template check_group<1>(q, C, K, K.sph, obs_of(a.P)) ? V_HIT : V_FREE;
}

// Persistent projection kernel: a grid of resident waves pulls configurations from a device
// work queue (atomic counter), one per lane, and refills a lane when its configuration ends.
// With a verdict array the collision check is fused: tree models walk the converged
// configuration's link bounds once more in FP32 and test them against the box around the
// obstacles, so a configuration with no link near the obstacles is FREE at once, and the others
// are queued for the exact check (k_check_lanes).
// Dynamic LDS: projection_lds.
template <class Model, class IO, class S, int MODE, bool TILE>
__device__ __forceinline__ void persistent_body(double* smem) {
  const ProjArgs& a0 = kernarg<ProjArgs>();
  const Consts& C = consts_of(a0.P);
  const int dof = dof_of<Model>(C);
  double* tiles = smem + kTabDoubles<Model>;
  const QLds q = q_lds<Model::D>(tiles);
  const QLds q0 = q_lds<Model::D>(tiles + (MODE == CYCLIC ? Model::D * blockDim.x : 0));  // cyclic: iterate at iteration start
  const auto tr = make_trig<Model, TILE>(smem, tiles + Model::D * blockDim.x);
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t n = a0.n;
  if (i < kCounters && a0.clear) a0.clear[i] = 0u;
  if (i >= a0.n_static) i = n;  // not part of the static share
  int k = 0;
  if (i < n) load_q<Model, IO>(a0, dof, i, q);
  constexpr bool fused = Model::broad_in_residual;
  // A converged lane that needs the broad phase waits (pending) until no lane of the wave is
  // still iterating or half the wave is waiting, so one FP32 walk serves all of them instead of
  // one walk per iteration count.
  bool pending = false;
  for (;;) {
    const bool active = i < n && !pending;
    const bool any_active = __any(active);
    if (!any_active && !__any(pending)) break;
    if (fused && (!any_active || __builtin_popcountll(uint64_t(__ballot(pending))) >= 32)) {
      const ProjArgs& a = kernarg<ProjArgs>();
      if (pending) {
        // broad phase on the converged configurations (an FP32 walk of the link bounds)
        a.verdict[i] = V_FREE;  // the exact check overwrites it with V_HIT if a link hits
        if (Model::broad_flag(q, C)) a.chk_idx[queue_q<Model>(q, a.chk_count, a.chk_q, a.defer_cap)] = int32_t(i);
        pending = false;
        i = a.n_static + int64_t(atomicAdd(a.counter, 1u));
        k = 0;
        if (i < n) load_q<Model, IO>(a, dof, i, q);
      }
      continue;
    }
    if (active) {
      double resid;
      int st = iteration<Model, S, MODE>(q, q0, tr, k, C, resid);
      const ProjArgs& a = kernarg<ProjArgs>();
      if (st == ST_DEFER) {
        const unsigned slot = queue_q<Model>(q, a.defer_count, a.defer_q, a.defer_cap);
        atomicAdd(a.P->fallback_counter, 1ull);
        a.defer_ik[2 * slot] = int32_t(i);
        a.defer_ik[2 * slot + 1] = k;
      } else if (st >= 0) {
        store_result<Model, IO>(a, dof, i, q, st, k, resid);
        if (a.verdict) {
          if constexpr (fused) {
            if (a.check && st == ST_CONVERGED) pending = true;  // the verdict comes with the wave's walk
            else a.verdict[i] = V_UNCHECKED;
          } else {
            a.verdict[i] = verdict_inline<Model>(q, C, a, st);
          }
        }
      }
      if ((st >= 0 || st == ST_DEFER) && !pending) {
        i = a.n_static + int64_t(atomicAdd(a.counter, 1u));
        k = 0;
        if (i < n) load_q<Model, IO>(a, dof, i, q);
      }
    }
  }
}


template <class Model, class S, int MODE>
constexpr int persist_waves_v = std::is_same<S, float>::value && MODE != CYCLIC ? PersistWaves<Model>::value : 1;

template <class Model, class IO, class S, int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(persist_waves_v<Model, S, MODE>)))
k_project_persistent(ProjArgs) {
  extern __shared__ double smem[];
  persistent_body<Model, IO, S, MODE, kTrigTile<Model, S, MODE>>(smem);
}

// Exact collision check of the configurations queued by k_project_persistent: one configuration per lane, a work item per
// 64 queued configurations, link and share of the clusters (grid-stride). A lane group per configuration walked the whole
// tree in every lane of the group and its wave ran the union of its groups' pair lists; here a link's chain is walked once
// per configuration, the boxes come by 64-byte scalar reads and a cluster's sixteen obstacles by vector reads of one address
// (64 of the 108 registers). Bound by instruction issue where most clusters are near, by the latency of those reads
// else: they stand before the sphere tests, so a cluster that no sphere reaches pays for them too.
// Before (groups of 4 lanes) and after, us: 65,536 humanoid configurations 26.5 -> 14.5, Digit 149 -> 98, 65,536 checked
// humanoid configurations near the shelves 156 -> 99, 4,000 dual-arm geodesics of 4 to 128 configurations 349 -> 86,
// 131,072 arm configurations 114 -> 17.2, 1,021 arm geodesics of 4 to 64 configurations 79 -> 31.
template <class Model>
__global__ void __launch_bounds__(256, 4) k_check_lanes(ProjArgs a) {
  __shared__ float4 slot_mem[4 * 64];  // launched with 256 threads
  const int64_t cnt = *a.chk_count;
  if (cnt == 0) return;
  constexpr int NL = Model::NGEO;
  const int lane = int(threadIdx.x) & 63;
  const int wpb = int(blockDim.x) >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  // (32 bits: the queue holds fewer than 2^31 configurations, 2^25 groups of at most 36 links)
  const uint32_t groups = uint32_t((cnt + 63) / 64), waves = gridDim.x * uint32_t(wpb);
  // Short queues: a link's clusters over up to 64 waves, as long as the launch has waves for it (trees: two rounds of
  // them, their links differ in work) and the scene clusters. Unsplit, a wave of a short queue tested every near cluster in
  // turn: 64 arm configurations among 200 scattered obstacles 31 us (17 split; a wave per configuration took 18), 365 of 512
  // humanoid configurations near the shelves 82 us (35; 44).
  const int n_clus = coll_of(a.P).n_clus;
  const uint32_t room = Model::D <= Model::kGatherMaxD ? waves : 2 * waves;
  int split = 0;  // log2
  while (split < 6 && (1 << split) < n_clus && ((groups * NL) << (split + 1)) <= room) ++split;
  uint64_t every = ~uint64_t(0);  // bits 0, 2^split, 2 * 2^split, ...
  if (split > 0) {
    every = 1;
    for (int k = 1 << split; k < 64; k *= 2) every |= every << k;
  }
  // Link by link from the last one (the chains' ends come late), so that a hit that one link finds spares its lane the links
  // after it: 65,536 humanoid configurations among 2,000 scattered obstacles 1,064 us group by group, 236 so.
  for (uint32_t item = blockIdx.x * uint32_t(wpb) + uint32_t(wave); item < ((groups * NL) << split); item += waves) {
    const uint32_t it = item >> split, part = item & ((1u << split) - 1);
    const uint32_t grp = it % groups;
    const int rank = NL - 1 - int(it / groups);
    const int64_t slot = int64_t(grp) * 64 + lane;
    const bool in = slot < cnt;
    const int64_t s = in ? slot : cnt - 1;
    const int64_t i = a.chk_idx[s];
    const bool live = in && a.verdict[i] != V_HIT;  // another item may have found a hit already
    if (!__any(live)) continue;
    const QGlob<double> q{a.chk_q, a.defer_cap, s, Model::D};
    Rig<float> X;
    const int l = Model::geo_frame(rank, q, consts_of(a.P), X);
    if (Model::link_hits(X, l, coll_of(a.P), obs_pad_of(a.P), live, slot_mem + wave * 64, every << part) && live)
      a.verdict[i] = V_HIT;  // queued as V_FREE
  }
}

// The same check with groups of L lanes per configuration: the autotuner's alternatives on long queues (chk_long, 2
// to 16 lanes), what a caller may force (chk_lanes, 2 to 64), and the launcher's choice where many obstacles are near.
// Every lane of a group walks the tree, and the group splits the sphere-obstacle tests of
// the (link, cluster) pairs it finds overlapping: smaller groups repeat fewer walks, but the lanes of
// a wave then run different pair lists and the wave runs their union, so the best size depends on
// the batch. 64 lanes: a wave per configuration, on short queues (at most `small` entries) each
// configuration's links split over up to 4 waves.
// Dynamic LDS: one configuration per lane group (D doubles each; a wave per configuration also
// keeps 64 candidate-sphere slots per wave), then the robot spheres and the obstacles (float4
// each); groups of 2 exist for families of at most kTailCheckLowLanesMaxD
// coordinates and run only where their staged configurations leave room for 4 workgroups per CU
// (min_lanes, from the launcher).
constexpr int kTailCheckLowLanesMaxD = 16;
constexpr size_t kTailCheckLdsBudget = 40 * 1024;  // a quarter of a CU's LDS

template <class Model, class IO, int L>
__device__ __forceinline__ void check_tail_body(const ProjArgs& a, int64_t small, int64_t cnt, double* smem) {
  constexpr int D = Model::D;
  const Consts& C = consts_of(a.P);
  const CollConsts& K = coll_of(a.P);
  int64_t parts = 1;
  if (L == 64 && cnt > 0) parts = small / cnt < 4 ? (small / cnt < 1 ? 1 : small / cnt) : 4;
  if (int64_t(blockIdx.x) * blockDim.x / L >= cnt * parts) return;  // no queued work for this block
  const QLdsU q{(QLdsU::LP)(smem + (threadIdx.x / L) * D)};
  // a wave per configuration: 64 candidate-sphere slots per wave after the configurations
  float4* slots = L == 64 ? reinterpret_cast<float4*>(smem + D * (blockDim.x / L)) + (threadIdx.x / 64) * 64 : nullptr;
  float4* sph = reinterpret_cast<float4*>(smem + D * (blockDim.x / L)) + (L == 64 ? (blockDim.x / 64) * 64 : 0);
  float4* obs = sph + K.n_sph;
  block_copy16(sph, K.sph, K.n_sph * 16);
  block_copy16(obs, obs_of(a.P), K.n_obs * 16);
  __syncthreads();
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  for (int64_t item = gid / L; item < cnt * parts; item += int64_t(gridDim.x) * blockDim.x / L) {
    const int64_t slot = item / parts;
    const int part = int(item - slot * parts);
    load_queued<Model, IO>(a.chk_q, a.defer_cap, slot, q);
    const bool hit = Model::template check_group<L>(q, C, K, sph, obs, part, int(parts), slots);
    if ((gid & (L - 1)) == 0 && hit) a.verdict[a.chk_idx[slot]] = V_HIT;  // queued as V_FREE
  }
}

template <class Model, class IO>
__global__ void __launch_bounds__(256) k_check_tail(ProjArgs a, int64_t small, int min_lanes) {
  extern __shared__ double smem[];
  const int64_t cnt = *a.chk_count;
  int L = a.chk_lanes != 0 ? a.chk_lanes : cnt <= small ? 64 : a.chk_long;
  if (L < min_lanes) L = min_lanes;
  if (L == 64) {
    check_tail_body<Model, IO, 64>(a, small, cnt, smem);
  } else if (L == 16) {
    check_tail_body<Model, IO, 16>(a, small, cnt, smem);
  } else if (L == 8) {
    check_tail_body<Model, IO, 8>(a, small, cnt, smem);
  } else if constexpr (Model::D <= kTailCheckLowLanesMaxD) {
    if (L == 2) check_tail_body<Model, IO, 2>(a, small, cnt, smem);
    else check_tail_body<Model, IO, 4>(a, small, cnt, smem);
  } else {
    check_tail_body<Model, IO, 4>(a, small, cnt, smem);
  }
}

// FP64 tail of the persistent variant: the configurations deferred by the FP32 kernel, one per
// lane (grid-stride over the queue), continued from their stored FP64 iterate with FP64 steps. Their
// collision check joins the persistent kernel's: broad phase here, flagged ones queued for
// the exact check (in-line, one lane each, it took half a millisecond on an arm batch of 2,089 such configurations).
// Dynamic LDS: projection_lds.
template <class Model, class IO, int MODE>
__global__ void __launch_bounds__(64) k_project_tail(ProjArgs a) {
  extern __shared__ double smem[];
  const int64_t cnt = *a.defer_count;
  if (int64_t(blockIdx.x) * blockDim.x >= cnt) return;  // no deferred work for this block
  const Consts& C = consts_of(a.P);
  const int dof = dof_of<Model>(C);
  double* tiles = smem + kTabDoubles<Model>;
  const QLds q = q_lds<Model::D>(tiles);
  const QLds q0 = q_lds<Model::D>(tiles + (MODE == CYCLIC ? Model::D * blockDim.x : 0));
  const auto tr = make_trig<Model, false>(smem, nullptr);
  for (int64_t slot = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; slot < cnt;
       slot += int64_t(gridDim.x) * blockDim.x) {
    const int64_t i = a.defer_ik[2 * slot];
    int k = a.defer_ik[2 * slot + 1];
    load_queued<Model, IO>(a.defer_q, a.defer_cap, slot, q);
    double resid;
    const int st = finish_fp64<Model, MODE>(q, q0, tr, k, C, resid);
    store_result<Model, IO>(a, dof, i, q, st, k, resid);
    if (a.verdict) {
      if constexpr (Model::broad_in_residual) {
        // as in the persistent kernel: the broad phase here, the exact check of flagged
        // configurations in the kernel launched after this one
        if (a.check && st == ST_CONVERGED) {
          a.verdict[i] = V_FREE;
          if (Model::broad_flag(q, C)) a.chk_idx[queue_q<Model>(q, a.chk_count, a.chk_q, a.defer_cap)] = int32_t(i);
        } else {
          a.verdict[i] = V_UNCHECKED;
        }
      } else {
        a.verdict[i] = verdict_inline<Model>(q, C, a, st);
      }
    }
  }
}

// Plain kernel: one launch per geodesic, one configuration per lane, projection and
// collision check in the same kernel, no work queues (the FP64 steps and the exact check of
// flagged configurations run in-line).
template <class Model, class IO, class S, int MODE>
__global__ void __launch_bounds__(64) k_project_plain(ProjArgs a) {
  extern __shared__ double smem[];
  const Consts& C = consts_of(a.P);
  const int dof = dof_of<Model>(C);
  double* tiles = smem + kTabDoubles<Model>;
  const QLds q = q_lds<Model::D>(tiles);
  const auto tr = make_trig<Model, kTrigTile<Model, S, MODE>>(smem, tiles + Model::D * blockDim.x);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  load_q<Model, IO>(a, dof, i, q);
  int k = 0, st;
  double resid;
  constexpr bool fused = Model::broad_in_residual;
  bool near = true;
  for (;;) {
    st = newton_iteration<Model, S, MODE == OUTER>(q, tr, k, C, resid);
    if (st >= 0) break;
    if (st == ST_DEFER) {  // same rule as the persistent variant: FP64 steps from here on
      atomicAdd(a.P->fallback_counter, 1ull);
      TrigFor<Model, false> live;
      if constexpr (StepOf<Model>::type::trig) live.tab = tr.tab;
      st = finish_fp64<Model, MODE>(q, q, live, k, C, resid);
      near = true;
      break;
    }
  }
  store_result<Model, IO>(a, dof, i, q, st, k, resid);
  if (a.verdict) {
    // same broad-phase rule as the persistent variant; the exact check runs in-line
    if (fused && a.check && st == ST_CONVERGED) near = Model::broad_flag(q, C);
    const bool skip = fused && a.check && st == ST_CONVERGED && !near;
    a.verdict[a.base + i] = skip ? uint8_t(V_FREE) : verdict_inline<Model>(q, C, a, st);
  }
}

struct CheckArgs {
  const DevProblem* P;
  int64_t n;
  const void* q;
  int64_t ld;
  const int8_t* status;  // nullable: check only CONVERGED configurations
  uint8_t* verdict;
  void* minsd;           // nullable
};

// check_batch: L lanes per configuration (L = 1 with the exhaustive minimum signed distance).
template <class Model, class IO, bool MINSD, int L>
__global__ void __launch_bounds__(256) k_check(CheckArgs a) {
  const Consts& C = consts_of(a.P);
  const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t i = gid / L;
  if (i >= a.n) return;  // whole groups leave together
  const bool lead = (gid & (L - 1)) == 0;
  if (a.status && a.status[i] != ST_CONVERGED) {
    if (lead) a.verdict[i] = V_UNCHECKED;
    return;
  }
  const QGlob<IO> q{static_cast<const IO*>(a.q), a.ld, i, dof_of<Model>(C)};
  if constexpr (MINSD) {
    static_assert(L == 1, "the exhaustive distance runs one lane per configuration");
    bool hit;
    float msd;
    Model::min_signed_distance(q, C, coll_of(a.P), obs_of(a.P), hit, msd);
    a.verdict[i] = hit ? V_HIT : V_FREE;
    st_io<IO>(a.minsd, i, double(msd));
  } else {
    const CollConsts& K = coll_of(a.P);
    const bool hit = Model::template check_group<L>(q, C, K, K.sph, obs_of(a.P));
    if (lead) a.verdict[i] = hit ? V_HIT : V_FREE;
  }
}

// check_batch without distances, first pass: one lane per configuration, the FP32 walk of the link
// bounds against the box around all obstacles (the same broad phase as the fused projection). A
// configuration with no link near the box is FREE; the others are marked FREE and queued (index,
// FP64 configuration) for the exact check, which overwrites the verdict of those it finds colliding.
template <class Model, class IO>
__global__ void __launch_bounds__(256) k_check_broad(CheckArgs a, unsigned* count, int32_t* idx, double* qbuf,
                                                     int64_t cap, unsigned* clear) {
  const Consts& C = consts_of(a.P);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i == 0 && clear) *clear = 0u;  // the count of the next call
  if (i >= a.n) return;
  if (a.status && a.status[i] != ST_CONVERGED) {
    a.verdict[i] = V_UNCHECKED;
    return;
  }
  const QGlob<IO> q{static_cast<const IO*>(a.q), a.ld, i, dof_of<Model>(C)};
  a.verdict[i] = V_FREE;
  if (Model::broad_flag(q, C)) idx[queue_q<Model>(q, count, qbuf, cap)] = int32_t(i);
}

struct VjpArgs {
  const DevProblem* P;
  int64_t n;
  const void* q;
  int64_t ld;
  const int8_t* status;
  const void* g;
  void* g_in;
  double cond_thr;
  unsigned int* defer_count;  // FP32 mode: configurations left to the FP64 tail kernel
  int32_t* defer_idx;
  unsigned int* clear;        // FP32 mode: the count of the next call, zeroed by the main kernel (nullptr: none)
};

// The VJP kernels keep the upstream gradient g of a lane in LDS, in the precision of the solve (a
// [D][64] tile per wave after the waves' FP64 iterate tiles), instead of in registers across the Gram
// and the factorisation, and stream g_in = g - J^T y out of the J^T y walk joint by joint.
template <class S>
struct GLds {
  using LP = __attribute__((address_space(3))) S*;
  LP base;
  __device__ __forceinline__ S operator[](int j) const { return base[j * 64]; }
  __device__ __forceinline__ void set(int j, S v) const { base[j * 64] = v; }
};
// The calling lane's column of g: smem holds blockDim.x / 64 FP64 iterate tiles, then as many g tiles.
template <int D, class S>
__device__ __forceinline__ GLds<S> g_lds(double* smem) {
  const int w = int(threadIdx.x) >> 6, l = int(threadIdx.x) & 63;
  S* base = reinterpret_cast<S*>(smem + (blockDim.x >> 6) * (D * 64)) + w * (D * 64) + l;
  return GLds<S>{(typename GLds<S>::LP)base};
}
// Sink of the J^T y walk: out[j] = acc stores g_in[j] = g[j] - acc (coordinates below dof).
template <class IO, class S>
struct VjpOut {
  IO* dst;  // g_in + i
  int64_t ld;
  GLds<S> g;
  int dof;
  struct Ref {
    const VjpOut* o;
    int j;
    __device__ __forceinline__ void operator=(S acc) const {
      if (j < o->dof) o->dst[int64_t(j) * o->ld] = IO(double(o->g[j]) - double(acc));
    }
  };
  __device__ __forceinline__ Ref operator[](int j) const { return Ref{this, j}; }
};

template <class Model, class IO, class S>
__device__ __forceinline__ void vjp_load(const VjpArgs& a, int dof, int64_t i, const QLds& q, const GLds<S>& g) {
  const IO* pq = static_cast<const IO*>(a.q) + i;
  const IO* pg = static_cast<const IO*>(a.g) + i;
  IO x[Model::D], y[Model::D];
  for (int c = 0; c < Model::D; ++c) {
    x[c] = c < dof ? *pq : IO(0);
    y[c] = c < dof ? *pg : IO(0);
    const int64_t ld = after(a.ld, c);
    pq += ld;
    pg += ld;
  }
  __builtin_amdgcn_sched_barrier(0);
  for (int c = 0; c < Model::D; ++c) {
    q.set(c, double(x[c]));
    g.set(c, S(y[c]));
  }
}

template <class IO>
__device__ __forceinline__ void vjp_fill(const VjpArgs& a, int dof, int64_t i, double v) {
  IO* p = static_cast<IO*>(a.g_in) + i;
  for (int c = 0; c < dof; ++c) p[int64_t(c) * a.ld] = IO(v);
}

// FP64 Gram, factorisation and projection for one lane: g_in = g - J^T (J J^T)^-1 J g (NaN where
// the FP64 factorisation fails).
template <class Model, class IO, class TR>
__device__ __forceinline__ void vjp64(const VjpArgs& a, int dof, int64_t i, const QLds& q, const GLds<double>& g, const TR& tr,
                                      const Consts& C) {
  constexpr int M = Model::M;
  using W = typename StepOf<Model>::type;
  typename W::template SD<double> sd;
  double G[M * (M + 1) / 2], v[M], invd[M], kappa;
  W::template step_data<double>(q, C, sd, tr);
  W::template gram_jv<double>(q, C, sd, tr, G, g, v);
  double maxd = 0.0;
  for (int r = 0; r < M; ++r) maxd = fmax(maxd, G[pidx(r, r)]);
  if (cholesky<Model, double>(G, invd, kappa, kFloorF64 * maxd, drop_bits<Model>(sd))) {
    chol_solve<Model, double>(G, invd, v);
    W::template jty<double>(q, C, sd, tr, v, VjpOut<IO, double>{static_cast<IO*>(a.g_in) + i, a.ld, g, dof});
  } else {
    vjp_fill<IO>(a, dof, i, __builtin_nan(""));
  }
}

// g_in = g - J^T (J J^T)^-1 J g at the converged configuration (J recomputed; the forward
// pass stores nothing beyond q and status). g_in = 0 for configurations that did not converge.
// In FP32 mode a lane whose factorisation fails or whose condition estimate exceeds the
// threshold is queued for k_vjp_tail, which redoes it in FP64.
// Dynamic LDS: the sine table, D * blockDim doubles (iterates), D * blockDim S (gradients).
template <class Model, class IO, class S>
__global__ void __launch_bounds__(64) k_vjp(VjpArgs a) {
  constexpr int D = Model::D, M = Model::M;
  extern __shared__ double smem[];
  constexpr bool f32 = std::is_same<S, float>::value;
  using W = typename StepOf<Model>::type;
  const Consts& C = consts_of(a.P);
  double* tiles = smem + kTabDoubles<Model>;
  const QLds q = q_lds<D>(tiles);
  const GLds<S> g = g_lds<D, S>(tiles);
  // the trig tile takes the iterate's place slot by slot: the one pass that reads the iterate writes it
  const auto tr = make_trig<Model, W::trig && f32>(smem, tiles);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if constexpr (f32)
    if (i == 0 && a.clear) *a.clear = 0u;
  if (i >= a.n) return;
  const int dof = dof_of<Model>(C);
  if (a.status[i] != ST_CONVERGED) {
    vjp_fill<IO>(a, dof, i, 0.0);
    return;
  }
  vjp_load<Model, IO, S>(a, dof, i, q, g);
  if constexpr (f32) {
    typename W::template SD<float> sd;
    float G[M * (M + 1) / 2], v[M], invd[M], kappa;
    W::template step_data<float>(q, C, sd, tr);
    W::template gram_jv<float>(q, C, sd, tr, G, g, v);
    if (cholesky<Model, float>(G, invd, kappa, kFloorF32, drop_bits<Model>(sd)) && double(kappa) <= a.cond_thr) {
      chol_solve<Model, float>(G, invd, v);
      W::template jty<float>(q, C, sd, tr, v, VjpOut<IO, float>{static_cast<IO*>(a.g_in) + i, a.ld, g, dof});
    } else {
      atomicAdd(a.P->fallback_counter, 1ull);
      a.defer_idx[atomicAdd(a.defer_count, 1u)] = int32_t(i);
    }
  } else {
    vjp64<Model, IO>(a, dof, i, q, g, tr, C);
  }
}

// FP64 redo of the VJPs queued by k_vjp (grid-stride over the queue).
// Dynamic LDS: the sine table, 2 * D * blockDim doubles (iterates, gradients).
template <class Model, class IO>
__global__ void __launch_bounds__(64) k_vjp_tail(VjpArgs a) {
  constexpr int D = Model::D;
  extern __shared__ double smem[];
  const int64_t cnt = *a.defer_count;
  if (int64_t(blockIdx.x) * blockDim.x >= cnt) return;  // no deferred work for this block
  const Consts& C = consts_of(a.P);
  const int dof = dof_of<Model>(C);
  double* tiles = smem + kTabDoubles<Model>;
  const QLds q = q_lds<D>(tiles);
  const GLds<double> g = g_lds<D, double>(tiles);
  const auto tr = make_trig<Model, false>(smem, nullptr);
  for (int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; s < cnt; s += int64_t(gridDim.x) * blockDim.x) {
    const int64_t i = a.defer_idx[s];
    vjp_load<Model, IO, double>(a, dof, i, q, g);
    vjp64<Model, IO>(a, dof, i, q, g, tr, C);
  }
}

// ---------------------------------------------------------------- exact VJP off the manifold
// The derivative of the projection map itself (not only of the projection at its output), by
// reverse mode through the Newton steps the forward pass took: with q_{k+1} = q_k - alpha J^T y,
// y = G^-1 F, G = J J^T + lambda I, a cotangent w of q_{k+1} pulls back to
//   w_k = w - alpha (J^T z + H(y.F) a - H(z.F) delta),   z = G^-1 J w, a = w - J^T z, delta = J^T y,
// where H(c.F) v is the Hessian-vector product of the scalar c.F, the directional derivative of its
// gradient J^T c along v (here by central differences of the analytic gradient in FP64). The output
// cotangent is first projected on the tangent space at q_K, which is what one more Newton step at
// the converged point does to it (the converged map's derivative there).
struct VjpxArgs {
  const DevProblem* P;
  int64_t n;
  const void* q_in;   // the forward pass's (unprojected) inputs
  int64_t ld;
  const int8_t* status;
  const int8_t* iters;  // the forward pass's step counts
  const void* g;
  void* g_in;
  double alpha, lambda, h_rel;
};

// A per-lane FP32 column of a [D][64] LDS tile.
struct FLds {
  using LP = __attribute__((address_space(3))) float*;
  LP base;
  __device__ __forceinline__ float operator[](int j) const { return base[j * 64]; }
  __device__ __forceinline__ void set(int j, float v) const { base[j * 64] = v; }
  __device__ __forceinline__ FLds fresh() const {
    FLds r = *this;
    asm volatile("" : "+v"(r.base));
    return r;
  }
};
// Sink of a J^T c walk that hands (j, value) to a callable.
template <class S, class Fn>
struct FnSink {
  Fn fn;
  struct Ref {
    const FnSink* o;
    int j;
    __device__ __forceinline__ void operator=(S acc) const { o->fn(j, acc); }
  };
  __device__ __forceinline__ Ref operator[](int j) const { return Ref{this, j}; }
};
template <class S, class Fn>
__device__ __forceinline__ FnSink<S, Fn> fn_sink(Fn fn) { return FnSink<S, Fn>{fn}; }
// The iterate moved along a unit direction: coordinate j is q_j + t u_j / |u|.
struct QShift {
  QLds q;
  FLds u;
  double t;  // step already divided by |u|
  __device__ __forceinline__ double at(int j) const { return q.at(j) + t * double(u[j]); }
  template <class U>
  __device__ __forceinline__ double at(int j, U dep) const { return q.at(j, dep) + t * double(u[j]); }
  __device__ __forceinline__ double get(int j) const { return q.get(j) + t * double(u[j]); }
  __device__ __forceinline__ QShift fresh() const { return QShift{q.fresh(), u.fresh(), t}; }
};

// FP64 Gram of J J^T + lambda I at q, factorised (and v = J g, where asked for); false when it is not positive definite.
template <class Model, bool WITH_V, class TR, class GV>
__device__ __forceinline__ bool gram64(const QLds& q, const TR& tr, const Consts& C, double lambda,
                                       typename StepOf<Model>::type::template SD<double>& sd, typename StepOf<Model>::type::Basis& bs,
                                       double* F, double* G, double* invd, GV g, double* v) {
  constexpr int M = Model::M;
  using W = typename StepOf<Model>::type;
  W::residual_basis(q, C, F, sd, bs, tr);
  if constexpr (WITH_V) W::template gram_jv<double>(q, C, sd, tr, G, g, v);
  else W::template gram<double>(q, C, sd, tr, G);
  if (lambda > 0.0) W::template add_lambda<double>(G, F, lambda, tr);
  double maxd = 0.0, kappa;
  for (int r = 0; r < M; ++r) maxd = fmax(maxd, G[pidx(r, r)]);
  return cholesky<Model, double>(G, invd, kappa, kFloorF64 * maxd, drop_bits<Model>(sd));
}

// k FP64 Newton steps from the input (replaying the forward pass's path); false on a failure. The loop runs as long as
// any lane has steps left, so the constants' scalar addresses stay wave-uniform over it.
template <class Model, class IO, class TR>
__device__ __forceinline__ bool replay(const VjpxArgs& a, int dof, int64_t i, int k, const QLds& q, const TR& tr, const Consts& C) {
  constexpr int M = Model::M;
  using W = typename StepOf<Model>::type;
  const IO* p = static_cast<const IO*>(a.q_in) + i;
  for (int c = 0; c < Model::D; ++c) q.set(c, c < dof ? double(p[int64_t(c) * a.ld]) : 0.0);
  bool ok = true;
  for (int s = 0; __any(ok && s < k); ++s) {
    if (!(ok && s < k)) continue;
    typename W::template SD<double> sd;
    typename W::Basis bs;
    double F[M], G[M * (M + 1) / 2], invd[M];
    if (!gram64<Model, false>(q, tr, C, a.lambda, sd, bs, F, G, invd, (const double*)nullptr, (double*)nullptr)) {
      ok = false;
      continue;
    }
    chol_solve<Model, double>(G, invd, F);
    const double al = a.alpha;
    // a walk has read coordinate j when it reports column j, so the update can go in place
    W::template jty<double>(q, C, sd, tr, F, fn_sink<double>([&](int j, double acc) { q.set(j, q.get(j) - al * acc); }));
  }
  return ok;
}

// Accumulate coef * (gradient of c.F at q + t u/|u|) into w (the FP64 cotangent tile: the two
// evaluations of a central difference add nearly cancelling terms of size |u| |grad| / 2h). c in the scene's rows.
// Rows that a lane may drop keep the base point's choice (base: the step data at q).
template <class Model, class TR>
__device__ __forceinline__ void grad_axpy(const QLds& q, const FLds& u, double t, const TR& tr, const double* c,
                                          double coef, const QLds& w,
                                          const typename StepOf<Model>::type::template SD<double>& base) {
  constexpr int M = Model::M;
  using W = typename StepOf<Model>::type;
  const Consts& C = consts_of(kernarg<VjpxArgs>().P);
  const QShift qs{q, u, t};
  typename W::template SD<double> sd;
  typename W::Basis bs;
  double F[M], y[M];
  W::residual_basis(qs, C, F, sd, bs, tr);
  W::freeze_rows(sd, base);
  for (int r = 0; r < M; ++r) y[r] = c[r];
  W::template change_rows<true>(bs, tr, y);
  W::template jty<double>(qs, C, sd, tr, y, fn_sink<double>([&](int j, double acc) { w.set(j, w.get(j) + coef * acc); }));
}

// Bound by FP64 instruction issue (one wave per SIMD, K <= 3 steps on the batches that use it: K (K - 1) / 2 + 1
// replayed steps and ten walks per reverse step). On walks that re-formed world-axis columns from the root, with the
// moments' prefix sums and 1.7 KB of spills per lane, it took 597 us for 18,530 humanoid configurations;
// on the leaf-to-root walks 411 us.
// Dynamic LDS: the sine table, per wave two FP64 tiles (iterate, cotangent) and an FP32 one (direction).
template <class Model, class IO>
__global__ void __launch_bounds__(64) k_vjp_exact(VjpxArgs a) {
  constexpr int D = Model::D, M = Model::M;
  using W = typename StepOf<Model>::type;
  extern __shared__ double smem[];
  const Consts& C = consts_of(a.P);
  // (FP32 gradients: the sines' last bit moves the differences below by 1e-12 of themselves, and costs 5 % of the kernel)
  const auto tr = make_trig<Model, false, std::is_same<IO, double>::value>(smem, nullptr);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const int dof = dof_of<Model>(C);
  IO* out = static_cast<IO*>(a.g_in) + i;
  if (a.status[i] != ST_CONVERGED) {
    for (int c = 0; c < dof; ++c) out[int64_t(c) * a.ld] = IO(0);
    return;
  }
  // tiles: the FP64 iterate and cotangent w (waves' tiles in turn), then the FP32 direction v (a, then delta)
  double* tiles = smem + kTabDoubles<Model>;
  const int nw = int(blockDim.x) >> 6, w0 = int(threadIdx.x) >> 6, l = int(threadIdx.x) & 63;
  const QLds q{(QLds::LP)(tiles + w0 * (D * 64) + l)};
  const QLds w{(QLds::LP)(tiles + (nw + w0) * (D * 64) + l)};
  float* fb = reinterpret_cast<float*>(tiles + 2 * nw * (D * 64));
  const FLds v{(FLds::LP)(fb + w0 * (D * 64) + l)};
  const int K = a.iters[i];
  bool ok = replay<Model, IO>(a, dof, i, K, q, tr, C);
  {
    const IO* pg = static_cast<const IO*>(a.g) + i;
    for (int c = 0; c < D; ++c) w.set(c, c < dof ? double(pg[int64_t(c) * a.ld]) : 0.0);
  }
  // w <- (I - J^+ J) w at q_K
  if (ok) {
    typename W::template SD<double> sd;
    typename W::Basis bs;
    double F[M], G[M * (M + 1) / 2], invd[M], z[M];
    ok = gram64<Model, true>(q, tr, C, 0.0, sd, bs, F, G, invd, w.fresh(), z);
    if (ok) {
      chol_solve<Model, double>(G, invd, z);
      W::template jty<double>(q, C, sd, tr, z, fn_sink<double>([&](int j, double acc) { w.set(j, w.get(j) - acc); }));
    }
  }
  for (int k = K - 1; k >= 0 && ok; --k) {
    ok = replay<Model, IO>(a, dof, i, k, q, tr, C);
    if (!ok) break;
    typename W::template SD<double> sd;
    typename W::Basis bs;
    double F[M], z[M];
    {
      double G[M * (M + 1) / 2], invd[M];
      ok = gram64<Model, true>(q, tr, C, a.lambda, sd, bs, F, G, invd, w.fresh(), z);
      if (!ok) break;
      chol_solve<Model, double>(G, invd, F);  // F <- y
      chol_solve<Model, double>(G, invd, z);  // z = G^-1 J w
    }
    const double al = a.alpha;
    // v <- a = w - J^T z, then w <- (1 - alpha) w + alpha a (= w - alpha J^T z)
    W::template jty<double>(q, C, sd, tr, z, fn_sink<double>([&](int j, double acc) {
      const double wj = w.get(j), aj = wj - acc;
      v.set(j, float(aj));
      w.set(j, (1.0 - al) * wj + al * aj);
    }));
    double qn = 1.0, vn = 0.0;
    for (int c = 0; c < D; ++c) {
      qn = fmax(qn, fabs(q.get(c)));
      vn += double(v[c]) * double(v[c]);
    }
    const double h = a.h_rel * qn;
    vn = sqrt(vn);
    // y and z in the scene's rows, which stay fixed where the gradients of y.F and z.F are differenced
    double ys[M], zs[M];
    for (int r = 0; r < M; ++r) {
      ys[r] = F[r];
      zs[r] = z[r];
    }
    W::template change_rows<false>(bs, tr, ys);
    W::template change_rows<false>(bs, tr, zs);
    // w -= alpha H(y.F) a: central difference of the gradient J^T y along a / |a|, times |a| / 2h
    if (vn > 0.0) {
      const double coef = al * vn / (2.0 * h);
      for (int sgn = 1; sgn >= -1; sgn -= 2) grad_axpy<Model>(q, v, sgn * h / vn, tr, ys, -sgn * coef, w, sd);
    }
    // v <- delta = J^T y, then w += alpha H(z.F) delta
    W::template jty<double>(q, C, sd, tr, F, fn_sink<double>([&](int j, double acc) { v.set(j, float(acc)); }));
    double dn = 0.0;
    for (int c = 0; c < D; ++c) dn += double(v[c]) * double(v[c]);
    dn = sqrt(dn);
    if (dn > 0.0) {
      const double coef = al * dn / (2.0 * h);
      for (int sgn = 1; sgn >= -1; sgn -= 2) grad_axpy<Model>(q, v, sgn * h / dn, tr, zs, sgn * coef, w, sd);
    }
  }
  for (int c = 0; c < dof; ++c) out[int64_t(c) * a.ld] = ok ? IO(w.at(c)) : IO(__builtin_nan(""));
}

// Diagnostic: residual (FP64) and dense Jacobian (step precision S) as the projection
// kernels compute them.
template <class Model, class IO, class S>
__global__ void __launch_bounds__(256) k_eval_fj(const DevProblem* Pp, int64_t n, const void* qv, int64_t ld, void* Fo, void* Jo) {
  constexpr int D = Model::D, M = Model::M;
  const Consts& P = consts_of(Pp);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int dof = P.dof, m = P.rows;
  const QGlob<IO> q{static_cast<const IO*>(qv), ld, i, dof};
  typename Model::template SD<double> sd64;
  double F[M];
  Model::template residual<double>(q, P, F, sd64);
  typename Model::template SD<S> sd;
  S Fs[M], J[M * D];
  Model::template residual<S>(q, P, Fs, sd);
  Model::template jacobian<S>(q, P, sd, J);
  for (int r = 0; r < M; ++r) {
    if (r >= m) continue;
    st_io<IO>(Fo, r * ld + i, F[r]);
    for (int c = 0; c < D; ++c)
      if (c < dof) st_io<IO>(Jo, (int64_t(r) * dof + c) * ld + i, double(J[r * D + c]));
  }
}

// Diagnostic: the condition estimate (max L_ii / min L_ii)^2 of J J^T + lambda I in precision S (+inf where the
// factorisation fails), in the rows of the passes W: the scene's own (Direct) or the projection kernels' (StepOf).
// Dynamic LDS: the sine table, D * blockDim doubles (iterates).
template <class Model, class IO, class S, class W>
__global__ void __launch_bounds__(64) k_eval_cond(const DevProblem* Pp, int64_t n, const void* qv, int64_t ld,
                                                  double lambda, void* kappa_out) {
  constexpr int D = Model::D, M = Model::M;
  extern __shared__ double smem[];
  const Consts& C = consts_of(Pp);
  const auto tr = make_trig<Model, false>(smem, nullptr);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int dof = dof_of<Model>(C);
  const QLds q = q_lds<D>(smem + kTabDoubles<Model>);
  const IO* p = static_cast<const IO*>(qv) + i;
  for (int c = 0; c < D; ++c) q.set(c, c < dof ? double(p[int64_t(c) * ld]) : 0.0);
  typename W::template SD<S> sd;
  S F[M], G[M * (M + 1) / 2], invd[M], kappa;
  W::template residual<S>(q, C, F, sd, tr);
  W::template gram<S>(q, C, sd, tr, G);
  if (lambda > 0.0) W::template add_lambda<S>(G, F, S(lambda), tr);
  S maxd = S(0);
  for (int r = 0; r < M; ++r) maxd = G[pidx(r, r)] > maxd ? G[pidx(r, r)] : maxd;
  const S floor = std::is_same<S, float>::value ? S(kFloorF32) : S(kFloorF64);
  const bool ok = cholesky<Model, S>(G, invd, kappa, floor * maxd, drop_bits<Model>(sd));
  st_io<IO>(kappa_out, i, ok ? double(kappa) : __builtin_huge_val());
}

}  // namespace mc
