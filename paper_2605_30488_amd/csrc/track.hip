// Ray-range tracking (Sec. III-A): each of n independent problems estimates the pose T_kf of a frame f
// relative to a keyframe k by minimising E_track(T_kf), the component-wise Huber cost of the whitened
// residual of eq. (1) over the frame-to-keyframe matches, with Levenberg-Marquardt damping (the tracker's
// form of eq. 7: (H + lambda diag H + eps_r I) tau = -g, T <- Exp(tau) T).
//
// Execution: the matches of every problem are gathered once into a match stream (the batched graph
// step's records: X_f[n], X_k[m], (C_k C_f)^(1/4)); then 1 + max_trials rounds run with no host
// synchronisation, each one launch for few segments and two otherwise: the stream reduction at every problem's trial pose (the graph step's
// residual / Jacobian / Huber / Hessian kernel, one edge per problem with the keyframe at the identity,
// so H = H_L and g = b_L), and the step, one block per problem, which sums the segment partials in
// a fixed order, takes the LM decision, solves the damped 7x7 system and writes the next trial pose.
// Problems that have stopped are skipped.
//
// The accept test compares E_track at two nearby poses. Near the optimum their difference falls below
// what a float32 evaluation resolves (each whitened ray residual is a difference of unit vectors over
// sigma_r = 0.003, so float32 rounding alone moves a pixel's cost by ~1e-4, and a 3k-pixel sum by ~1e-3
// while the true decrease per step reaches 1e-8): a float32 test rejects good steps there, inflates the
// damping and stops short of the optimum. The reduction therefore also evaluates each segment's cost in
// float64 (from the stored values and the float64 trial pose), and only that cost enters the decision;
// H and g stay float32.
#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "common.hpp"
#include "internal.hpp"
#include "sim3.hpp"
#include "track_step.hpp"

namespace ds3 {

size_t track_state_bytes() { return sizeof(TrackState); }

// One block per problem (see track_step).
__global__ __launch_bounds__(kStepThreads) void k_track_step(const EdgeDev* __restrict__ edges,
                                                             const float* __restrict__ partials,
                                                             const double* __restrict__ cost64, TrackIo io, int phase) {
  const int p = blockIdx.x;
  if (phase > 0 && io.done[p]) return;
  track_step<false>(edges[p], p, partials, cost64, io, phase);
}

// Initial transform of every problem (float32 and float64 copies of T_io) for the phase-0 reduction.
__global__ void k_track_init(const double* __restrict__ T_io, int n, EdgeXf* __restrict__ xf,
                             double* __restrict__ xf64, int32_t* __restrict__ done,
                             TrackState* __restrict__ states) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  Sim3 T = sim3_load(T_io + 8 * int64_t(p));
  quat_normalize(T.q);
  write_xf(T, xf + p, xf64 + 12 * int64_t(p));
  done[p] = 0;
  states[p].ticket = 0;
}

int launch_track_init(const TrackIo& io, int n, hipStream_t s) {
  if (n <= 0) return DS3_OK;
  hipLaunchKernelGGL(k_track_init, dim3((n + 63) / 64), dim3(64), 0, s, io.T_io, n, io.xf, io.xf64, io.done, io.states);
  return check_hip(hipGetLastError(), "k_track_init");
}

int launch_track_step(const EdgeDev* edges, int n, const float* partials, const double* cost64, const TrackIo& io,
                      int phase, hipStream_t s) {
  if (n <= 0) return DS3_OK;
  hipLaunchKernelGGL(k_track_step, dim3(n), dim3(kStepThreads), 0, s, edges, partials, cost64, io, phase);
  return check_hip(hipGetLastError(), "k_track_step");
}

}  // namespace ds3

// ------------------------------------------------------------------------------------------------------
// C ABI
// ------------------------------------------------------------------------------------------------------
namespace ds3 {

constexpr int kTrackPPT = 16;  // segment = 4096 frame pixels

// Calls with at most this many segments run each round as one launch of three blocks per segment (k_track_round).
// us per call, one launch against two (float32; bfloat16 agrees within 10%, but for 498 to 464 at five frames):
//   512 x 384 frames (48 segments): 1 frame 338 to 435, 3 frames 374 to 449, 4: 403 to 445, 5: 417 to 451, 8: 527 to 498
//   128 x 96 frames (3 segments): 1 frame 308 to 411, 32 frames 370 to 446, 53: 383 to 448, 64: 434 to 448, 85: 561 to 454
//   64 x 48 frames (1 segment): 1 frame 283 to 332, 96 frames 357 to 392, 160: 338 to 401, 192: 458 to 406, 256: 437 to 411
// Up to 170 segments, two blocks per CU, one launch gains with frames of any size. Past that the records that each role
// reads again begin to cost more than the launch: whole frames, as online tracking has them, still gain up to about this
// limit (a block per CU in the two-launch form's reduction), many short ones lose 3 to 20% there.
constexpr int kRoundItems = 256;

struct TrackBuffers {
  EdgeDev* edges;
  WorkItem* items;
  EdgeXf* xf;
  double* xf64;
  float* partials;
  double* cost64;
  void* stream;
  int32_t* seg_count;
  void* states;
  int32_t* done;
};

static int track_topology(int n, const ds3_track_problem* probs, std::vector<EdgeDev>& edges,
                          std::vector<WorkItem>& items) {
  if (n < 0 || (n > 0 && !probs)) return fail(DS3_EINVAL, "track: bad problem table");
  const int seg = kReduceThreads * kTrackPPT;
  edges.resize(n);
  items.clear();
  int64_t tiles = 0;
  for (int p = 0; p < n; ++p) {
    const ds3_track_problem& q = probs[p];
    const ds3_image& K = q.keyframe;
    const ds3_image& F = q.frame;
    if (K.H <= 0 || K.W <= 0 || F.H <= 0 || F.W <= 0 || K.px_offset < 0 || F.px_offset < 0 || q.idx_offset < 0 ||
        int64_t(K.H) * K.W > INT32_MAX || int64_t(F.H) * F.W > INT32_MAX)
      return fail(DS3_EINVAL, "track: bad problem " + std::to_string(p));
    EdgeDev D;
    D.off_i = K.px_offset;
    D.off_j = F.px_offset;
    D.idx_off = q.idx_offset;
    D.npx_i = K.H * K.W;
    D.npx_j = F.H * F.W;
    D.i = 0;
    D.j = 0;
    D.tile0 = int32_t(tiles);
    D.n_tiles = (D.npx_j + seg - 1) / seg;
    for (int t = 0; t < D.n_tiles; ++t) items.push_back(WorkItem{p, t});
    tiles += D.n_tiles;
    if (tiles > INT32_MAX / seg) return fail(DS3_EINVAL, "track: too many frame pixels for one call");
    edges[p] = D;
  }
  return DS3_OK;
}

static size_t carve_track(void* base, int n, int tiles, ds3_dtype dt, TrackBuffers& B) {
  Carver c(base);
  const size_t seg = size_t(kReduceThreads) * kTrackPPT;
  B.edges = c.take<EdgeDev>(std::max(n, 1));
  B.items = c.take<WorkItem>(std::max(tiles, 1));
  B.xf = c.take<EdgeXf>(std::max(n, 1));
  B.xf64 = c.take<double>(size_t(std::max(n, 1)) * 12);
  B.partials = c.take<float>(size_t(std::max(tiles, 1)) * kPartial);
  B.cost64 = c.take<double>(std::max(tiles, 1));
  B.stream = c.take<char>(size_t(std::max(tiles, 1)) * seg * stream_record_bytes(dt));
  B.seg_count = c.take<int32_t>(std::max(tiles, 1));
  B.states = c.take<char>(size_t(std::max(n, 1)) * track_state_bytes());
  B.done = c.take<int32_t>(std::max(n, 1));
  return c.used;
}

// Static scratch of ds3_track_noalloc: a file-scope device array, one copy per GPU, held until the
// process ends. Host code reaches it only through the address hipGetSymbolAddress returns for the
// current device (the array's own name is a host-side stand-in, not a device address).
constexpr size_t kTrackScratchBytes = size_t(DS3_TRACK_SCRATCH_BYTES);
static __device__ __align__(256) char scratch[kTrackScratchBytes];

static int track_scratch(void** out) {
  static std::mutex mu;
  static std::vector<void*> addr;
  int dev = 0;
  DS3_TRY_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(mu);
  if (int(addr.size()) <= dev) addr.resize(dev + 1, nullptr);
  if (!addr[dev]) {
    void* p = nullptr;
    DS3_TRY_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    addr[dev] = p;
  }
  *out = addr[dev];
  return DS3_OK;
}

static int track_impl(const void* arena, ds3_dtype dtype, const ds3_track_problem* probs, int32_t n,
                      const int32_t* idx_arena, const ds3_gn_params* gn, const ds3_track_params* tp, double* T,
                      double* cost_out, int32_t* trials_out, int32_t* status_out, ds3_timer* reduce_timer,
                      void* workspace, size_t ws_bytes, void* stream) {
  if (n < 0) return fail(DS3_EINVAL, "track: n < 0");
  if (n == 0) return DS3_OK;
  if (!arena || !idx_arena || !gn || !tp || !T || !cost_out || !trials_out || !workspace)
    return fail(DS3_EINVAL, "track: null pointer");
  if (dtype != DS3_F32 && dtype != DS3_BF16) return fail(DS3_ENOTSUP, "track: dtype");
  if ((reinterpret_cast<uintptr_t>(arena) & 15) != 0) return fail(DS3_EINVAL, "track: arena must be 16 B aligned");
  if (!(gn->sigma_ray > 0) || !(gn->sigma_dist > 0) || !(gn->huber_k > 0) || gn->max_attempts < 1 ||
      gn->max_attempts > 16)
    return fail(DS3_EINVAL, "track: bad graph-step constants");
  if (gn->K) return fail(DS3_ENOTSUP, "track: no calibrated mode (K must be NULL)");
  if (tp->max_trials < 0 || tp->max_trials > 1000 || !(tp->lambda0 >= 0) || !(tp->lambda_up >= 1) ||
      !(tp->lambda_down > 0) || !(tp->lambda_down <= 1) || !(tp->lambda_min >= 0) || !(tp->step_tol >= 0))
    return fail(DS3_EINVAL, "track: bad LM schedule");
  std::vector<EdgeDev> edges;
  std::vector<WorkItem> items;
  DS3_TRY(track_topology(n, probs, edges, items));
  const int tiles = int(items.size());
  TrackBuffers B;
  if (ws_bytes < carve_track(nullptr, n, tiles, dtype, B)) return fail(DS3_ENOSPACE, "track: workspace too small");
  carve_track(workspace, n, tiles, dtype, B);
  hipStream_t s = static_cast<hipStream_t>(stream);
  TableUpload u;
  u.add(B.edges, edges);
  u.add(B.items, items);
  DS3_TRY(u.flush(s));
  const int seg = kReduceThreads * kTrackPPT;
  const GnConst c = make_gn_const(*gn);
  TrackConst tc;
  tc.lambda0 = tp->lambda0;
  tc.lambda_min = tp->lambda_min;
  tc.lambda_up = tp->lambda_up;
  tc.lambda_down = tp->lambda_down;
  tc.step_tol = tp->step_tol;
  tc.eps0 = gn->eps0;
  tc.eps_mult = gn->eps_mult;
  tc.max_trials = tp->max_trials;
  tc.attempts = gn->max_attempts;
  const TrackIo io{static_cast<TrackState*>(B.states), B.done, B.xf, B.xf64, T, cost_out, trials_out, status_out, tc};
  DS3_TRY(launch_gather_stream(dtype, arena, B.edges, B.items, tiles, idx_arena, seg, B.stream, B.seg_count, s));
  DS3_TRY(launch_track_init(io, n, s));
  for (int phase = 0; phase <= tp->max_trials; ++phase) {
    if (tiles <= kRoundItems && !reduce_timer) {
      DS3_TRY(launch_track_round(dtype, B.stream, B.seg_count, B.edges, B.items, tiles, seg, B.partials, c, B.cost64, io,
                                 phase, s));
      continue;
    }
    const bool timed = reduce_timer && phase == 0;
    if (timed) DS3_TRY(timer_record(reduce_timer, true, s));
    DS3_TRY(launch_reduce_stream(dtype, 2, B.stream, B.seg_count, B.edges, B.items, tiles, B.xf, seg, B.partials,
                                 c, B.done, s, B.xf64, B.cost64));
    if (timed) DS3_TRY(timer_record(reduce_timer, false, s));
    DS3_TRY(launch_track_step(B.edges, n, B.partials, B.cost64, io, phase, s));
  }
  return DS3_OK;
}


}  // namespace ds3

using namespace ds3;

extern "C" {

void ds3_default_track_params(ds3_track_params* p) {
  if (!p) return;
  p->lambda0 = 1e-4;
  p->lambda_min = 1e-9;
  p->lambda_up = 10.0;
  p->lambda_down = 0.1;
  p->max_trials = 20;
  p->step_tol = 1e-7;
}

size_t ds3_track_workspace_bytes(int32_t n, const ds3_track_problem* probs, ds3_dtype dtype) {
  std::vector<EdgeDev> edges;
  std::vector<WorkItem> items;
  if (n <= 0 || track_topology(n, probs, edges, items) != DS3_OK) return 0;
  TrackBuffers B;
  return carve_track(nullptr, n, int(items.size()), dtype, B);
}

int ds3_track(const void* arena, ds3_dtype dtype, const ds3_track_problem* probs, int32_t n,
              const int32_t* idx_arena, const ds3_gn_params* gn, const ds3_track_params* tp, double* T,
              double* cost_out, int32_t* trials_out, int32_t* status_out, ds3_timer* reduce_timer,
              void* workspace, size_t ws_bytes, void* stream) {
  return track_impl(arena, dtype, probs, n, idx_arena, gn, tp, T, cost_out, trials_out, status_out, reduce_timer,
                    workspace, ws_bytes, stream);
}

int ds3_track_noalloc(const void* arena, ds3_dtype dtype, const ds3_track_problem* probs, int32_t n,
                      const int32_t* idx_arena, const ds3_gn_params* gn, const ds3_track_params* tp, double* T,
                      double* cost_out, int32_t* trials_out, int32_t* status_out, void* stream) {
  if (n < 0) return fail(DS3_EINVAL, "track_noalloc: n < 0");
  if (n == 0) return DS3_OK;
  std::vector<EdgeDev> edges;
  std::vector<WorkItem> items;
  DS3_TRY(track_topology(n, probs, edges, items));
  TrackBuffers B;
  const size_t need = carve_track(nullptr, n, int(items.size()), dtype, B);
  if (need > kTrackScratchBytes)
    return fail(DS3_ENOSPACE, "track_noalloc: these problems need " + std::to_string(need) +
                                  " bytes of scratch; the static scratch holds " +
                                  std::to_string(kTrackScratchBytes) + " (DS3_TRACK_SCRATCH_BYTES)");
  void* ws = nullptr;
  DS3_TRY(track_scratch(&ws));
  return track_impl(arena, dtype, probs, n, idx_arena, gn, tp, T, cost_out, trials_out, status_out, nullptr, ws,
                    kTrackScratchBytes, stream);
}

}  // extern "C"
