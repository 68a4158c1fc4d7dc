// One LM step of a tracking problem (Sec. III-A), run by one block of kStepThreads threads after the reduction has left
// the sums of the problem's segments: used by the step's own launch and by the round that runs it in its last block.
#pragma once

#include "common.hpp"
#include "internal.hpp"
#include "sim3.hpp"

namespace ds3 {

struct TrackState {
  double T[8];    // kept pose
  double Tt[8];   // trial pose the last reduction evaluated
  double tau[7];  // the step that produced Tt
  double H[28];   // upper triangle of H at T (row-major pairs r <= c)
  double b[7];
  double E;       // E_track at T
  double lam;
  int32_t trials, status, count;
  int32_t ticket;  // blocks of the current round that have stored their sums (k_track_round); 0 between rounds
};
static_assert(sizeof(TrackState) % sizeof(double) == 0, "copied as doubles");

// What a step reads and writes besides the problem's segments.
struct TrackIo {
  TrackState* states;
  int32_t* done;
  EdgeXf* xf;
  double* xf64;
  double* T_io;
  double* cost_out;
  int32_t* trials_out;
  int32_t* status_out;
  TrackConst tc;
};

__device__ constexpr int track_hidx(int r, int c) { return r * 7 - (r * (r - 1)) / 2 + (c - r); }

// (H + lam diag H + eps_r I) tau = -b by Cholesky with the epsilon ladder; returns the attempt used or -1
// (tau = 0) when every attempt fails (a non-positive or non-finite pivot). Fully unrolled, so the factor stays in
// registers (indexed by loops it lived in scratch memory).
__device__ inline int solve7(const double* Hin, const double* bin, double lam, double eps0, double mult, int attempts,
                             double* tau) {
  double H[28], b[7];
#pragma unroll
  for (int k = 0; k < 28; ++k) H[k] = Hin[k];
#pragma unroll
  for (int k = 0; k < 7; ++k) b[k] = bin[k];
  double eps = eps0;
#pragma unroll 1
  for (int r = 0; r < attempts; ++r, eps *= mult) {
    double L[49];
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) L[7 * i + j] = H[track_hidx(j, i)];
#pragma unroll
    for (int i = 0; i < 7; ++i) L[8 * i] += lam * H[track_hidx(i, i)] + eps;
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      double d = L[8 * j];
#pragma unroll
      for (int k = 0; k < j; ++k) d -= L[7 * j + k] * L[7 * j + k];
      if (!(d > 0.0) || !isfinite(d)) {
        ok = false;
        break;
      }
      const double ljj = sqrt(d);
      L[8 * j] = ljj;
#pragma unroll
      for (int i = j + 1; i < 7; ++i) {
        double v = L[7 * i + j];
#pragma unroll
        for (int k = 0; k < j; ++k) v -= L[7 * i + k] * L[7 * j + k];
        L[7 * i + j] = v / ljj;
      }
    }
    if (!ok) continue;
    double y[7], x[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      double v = -b[i];
#pragma unroll
      for (int k = 0; k < i; ++k) v -= L[7 * i + k] * y[k];
      y[i] = v / L[8 * i];
    }
#pragma unroll
    for (int i = 6; i >= 0; --i) {
      double v = y[i];
#pragma unroll
      for (int k = i + 1; k < 7; ++k) v -= L[7 * k + i] * x[k];
      x[i] = v / L[8 * i];
    }
#pragma unroll
    for (int i = 0; i < 7; ++i) tau[i] = x[i];
    return r;
  }
  for (int i = 0; i < 7; ++i) tau[i] = 0.0;
  return -1;
}

// The trial transform for the next reduction: float32 (H, g) and float64 (the cost of the accept test).
__device__ inline void write_xf(const Sim3& T, EdgeXf* xf, double* xf64) {
  double R[9];
  quat_to_mat(T.q, R);
  EdgeXf X;
  for (int r = 0; r < 3; ++r) {
    for (int c = 0; c < 3; ++c) {
      xf64[3 * r + c] = T.s * R[3 * r + c];
      X.m[3 * r + c] = float(T.s * R[3 * r + c]);
    }
    xf64[9 + r] = T.t[r];
    X.m[9 + r] = float(T.t[r]);
  }
  for (int k = 0; k < 4; ++k) X.pad[k] = 0.0f;
  *xf = X;
}

constexpr int kStepThreads = 256;
constexpr int kStepTiles = 64;  // segment partials staged in LDS at a time

// phase 0: the partials hold the sums at the initial poses (T_io); later phases: at the trial poses. The segments' sums
// are staged through LDS with every load in flight and added in segment order; the state is read and written by
// the block's threads side by side; one thread solves and moves the pose. Bound by that thread's chain of float64
// operations: 10.8 us for a problem of 48 segments. Each thread loading its sums segment by segment, the cost in one
// thread load by load, and the factor in scratch memory took 29 us.
// SAME_LAUNCH: the sums were published by other blocks of this launch, so they are read at device scope.
template <bool SAME_LAUNCH>
__device__ inline void track_step(const EdgeDev& E, int p, const float* partials, const double* cost64,
                                  const TrackIo& io, int phase) {
  __shared__ __align__(16) float stage[kStepTiles * kPartial];
  __shared__ double stage64[kStepTiles];
  __shared__ double S[37];
  __shared__ double Ecost;
  __shared__ TrackState st;
  const int t = threadIdx.x;
  constexpr int kStateWords = sizeof(TrackState) / sizeof(double);
  TrackState* g = io.states + p;
  if (phase > 0 && t >= 128 && t < 128 + kStateWords)
    reinterpret_cast<double*>(&st)[t - 128] = reinterpret_cast<const double*>(g)[t - 128];
  double s = 0.0, c = 0.0;
  for (int k0 = 0; k0 < E.n_tiles; k0 += kStepTiles) {
    const int m = min(kStepTiles, E.n_tiles - k0);
    if constexpr (SAME_LAUNCH) {
      // 8 B at a time, every load of the thread before its first use
      const auto* src = reinterpret_cast<const unsigned long long*>(partials + int64_t(E.tile0 + k0) * kPartial);
      constexpr int kLoads = kStepTiles * (kPartial / 2) / kStepThreads;
      static_assert(kLoads * kStepThreads == kStepTiles * (kPartial / 2), "whole rounds of loads");
      unsigned long long v[kLoads];
      double c64 = 0.0;
#pragma unroll
      for (int u = 0; u < kLoads; ++u)
        if (u * kStepThreads + t < m * (kPartial / 2))
          v[u] = __hip_atomic_load(src + u * kStepThreads + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (t < m) c64 = __hip_atomic_load(cost64 + E.tile0 + k0 + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int u = 0; u < kLoads; ++u)
        if (u * kStepThreads + t < m * (kPartial / 2))
          reinterpret_cast<unsigned long long*>(stage)[u * kStepThreads + t] = v[u];
      if (t < m) stage64[t] = c64;
    } else {
      const float4* src = reinterpret_cast<const float4*>(partials + int64_t(E.tile0 + k0) * kPartial);
      for (int q = t; q < m * (kPartial / 4); q += kStepThreads) reinterpret_cast<float4*>(stage)[q] = src[q];
      if (t < m) stage64[t] = cost64[E.tile0 + k0 + t];
    }
    __syncthreads();
    if (t < 37) {
#pragma unroll 8
      for (int k = 0; k < m; ++k) s += double(stage[k * kPartial + t]);
    }
    if (t == kWave) {  // the float64 cost, another wave than the sums'
#pragma unroll 8
      for (int k = 0; k < m; ++k) c += stage64[k];
    }
    __syncthreads();
  }
  if (t < 37) S[t] = s;
  if (t == kWave) Ecost = c;
  __syncthreads();
  // the decision, the same in every thread
  const TrackConst& tc = io.tc;
  const double E_new = Ecost;
  const bool accept = phase == 0 || E_new < st.E;
  bool stop = false;
  if (phase > 0) {
    if (accept) {  // keep the trial pose and its linearisation
      double m = 0.0;
      for (int k = 0; k < 7; ++k) m = fmax(m, fabs(st.tau[k]));
      if (m < tc.step_tol) stop = true;
    }
    if (st.trials + 1 >= tc.max_trials) stop = true;
  }
  __syncthreads();
  if (accept) {
    if (t < 28) st.H[t] = S[t];
    if (t >= 28 && t < 35) st.b[t - 28] = S[t];
    if (t >= kWave && t < kWave + 8) st.T[t - kWave] = phase == 0 ? io.T_io[8 * int64_t(p) + t - kWave] : st.Tt[t - kWave];
  }
  if (t == 128) {
    st.ticket = 0;
    if (phase == 0) {
      st.trials = 0;
      st.status = 0;
      st.lam = tc.lambda0;
    } else {
      st.trials += 1;
      st.lam = accept ? fmax(st.lam * tc.lambda_down, tc.lambda_min) : st.lam * tc.lambda_up;
    }
    if (accept) {
      st.E = E_new;
      st.count = int32_t(S[36] + 0.5);
    }
  }
  __syncthreads();
  if (t == 0) {
    if (!stop) {
      double tau[7];
      st.status = solve7(st.H, st.b, st.lam, tc.eps0, tc.eps_mult, tc.attempts, tau);
      // The pose is computed as from stored values: without this the compiler fuses the last products of the solve into
      // the first sums of the exponential, and decisions between nearly equal costs rest on the last bits.
#pragma unroll
      for (int k = 0; k < 7; ++k) asm volatile("" : "+v"(tau[k]));
      for (int k = 0; k < 7; ++k) st.tau[k] = tau[k];
      const Sim3 Tt = sim3_mul(sim3_exp(tau), sim3_load(st.T));
      Sim3 Tn = Tt;
      quat_normalize(Tn.q);
      sim3_store(Tn, st.Tt);
      write_xf(Tn, io.xf + p, io.xf64 + 12 * int64_t(p));
    } else {
      io.done[p] = 1;
    }
    io.cost_out[p] = st.E;
    io.trials_out[p] = st.trials;
    if (io.status_out) io.status_out[p] = st.status;
  }
  __syncthreads();
  if (t < 8) io.T_io[8 * int64_t(p) + t] = st.T[t];
  if (t >= 128 && t < 128 + kStateWords)
    reinterpret_cast<double*>(g)[t - 128] = reinterpret_cast<const double*>(&st)[t - 128];
}

}  // namespace ds3
