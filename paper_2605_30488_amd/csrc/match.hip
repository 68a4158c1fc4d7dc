// Projective ray matching (Sec. III-A "Learned geometry": p* = argmin_p |psi([X_ref]_p) - psi(x)|^2)
// and bidirectional verification with the nu gate (Sec. III-B).
//
// Per query pixel: Levenberg-Marquardt over the continuous reference pixel p on the bilinear interpolant
// of the reference ray image psi(X_ref) (not renormalised), started at the query's own pixel scaled to
// the reference grid; a trial step is accepted iff it lowers |s(p) - psi(x)|^2 (damping / 10, floored),
// otherwise the damping grows x10; stop after max_iters trial steps or a trial step (accepted or not)
// below step_tol_px. idx = round(p*) (ties up). Valid iff no hole was touched, the final angular residual is
// within ang_tol_px * min(|ds/du|, |ds/dv|) and the range agrees within range_rel_tol. The mutual check
// keeps pixel n of j iff its match m in i maps back within a Chebyshev radius of n.
//
// The reference ray image is built once per keyframe (psi as 12 bytes, NaN in holes, and |X| apart) so each LM
// sample reads 24 bytes of two rows. Batched launches walk (direction, strip) items laid end to end, an eighth
// per XCD (block b runs on XCD b mod 8), with the directions of one reference side by side, keeping that
// reference ray image in one L2.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "match_internal.hpp"

namespace ds3 {

// Ray image of every pixel: psi as three consecutive floats (NaN for a hole), |X| as a plain array (0 for a hole) and,
// when conf is given, its confidence as a plain float array (the mutual check then reads 4 B per pixel instead of a 16 B
// or 8 B xyzc entry). The pixels are n0 of arena and the others of arena1.
template <int DT>
__global__ void k_raymap(const void* __restrict__ arena, const void* __restrict__ arena1, int64_t n0, int64_t n,
                         float* __restrict__ rays, float* __restrict__ range, float* __restrict__ conf) {
  int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (; k < n; k += stride) {
    float4 X = k < n0 ? Px<DT>::load(arena, k) : Px<DT>::load(arena1, k - n0);
    if (conf) conf[k] = X.w;
    float d2 = fmaf(X.x, X.x, fmaf(X.y, X.y, X.z * X.z));
    float3 r = make_float3(__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf(""));
    float d = 0.f;
    if (finite3(X.x, X.y, X.z) && d2 > 1e-18f) {
      float rd = 1.0f / sqrtf(d2);
      d = sqrtf(d2);
      r = make_float3(X.x * rd, X.y * rd, X.z * rd);
    }
    rays[3 * k] = r.x;
    rays[3 * k + 1] = r.y;
    rays[3 * k + 2] = r.z;
    range[k] = d;
  }
}

int launch_raymap(const void* arena, int64_t n0, const void* arena1, int64_t n1, ds3_dtype dt, float* rays, float* range,
                  float* conf, hipStream_t s) {
  const int64_t n = n0 + n1;
  if (n <= 0) return DS3_OK;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (dt == DS3_F32)
    hipLaunchKernelGGL(k_raymap<DS3_F32>, dim3(blocks), dim3(256), 0, s, arena, arena1, n0, n, rays, range, conf);
  else
    hipLaunchKernelGGL(k_raymap<DS3_BF16>, dim3(blocks), dim3(256), 0, s, arena, arena1, n0, n, rays, range, conf);
  return check_hip(hipGetLastError(), "k_raymap");
}

// The last cell a query sampled, as differences: a and c are the upper and the lower left texel minus the query's target
// ray, ab and cd the steps to the right texels (of the texels minus the target ray). A trial that stays in the same cell
// (the common case once the steps are sub-pixel, and for every damped retry that moves a little) reuses them instead of
// gathering again. Interpolating the differences gives the residual s(p) - psi(x) directly: neighbouring rays differ from
// the target by about a pixel's angle, so their differences are nearly exact in float32 and the residual keeps its
// relative precision down to the optimum, where s(p) and psi(x) agree to six digits. (Interpolating the rays first and
// subtracting afterwards loses those digits: the cost then stops decreasing at steps of about 1e-4 px.) A hole is a
// texel of NaN, so every sample of its four cells is NaN and no flag is kept.
template <bool BIG>
struct Cell {
  using Coord = typename std::conditional<BIG, int, float>::type;
  Coord u0, v0;  // whole numbers
  float a[3], ab[3], c[3], cd[3];
};

// The ray image of one reference. 12-byte rays: a row's two texels are 24 bytes, read as 16 + 8.
struct RayImage {
  const float* rays;
  const float* range;
  int H, W;
};

// BIG: more than 2^24 pixels, where a pixel's index is no longer exact in float32.
template <bool BIG>
__device__ inline typename Cell<BIG>::Coord cell_origin(float u, int n) {
  if constexpr (BIG) return max(min(int(floorf(u)), n - 2), 0);
  else return fminf(floorf(u), float(n - 2));
}

// target(k, texel): the texel's component k minus the target ray's.
template <bool BIG, class F>
__device__ inline void fetch_cell(const RayImage& R, typename Cell<BIG>::Coord u0, typename Cell<BIG>::Coord v0,
                                  F target, Cell<BIG>& C) {
  float p[6], q[6];
  if constexpr (BIG) {
    const float* at = R.rays + 3 * (int64_t(v0) * R.W + u0);
    __builtin_memcpy(p, __builtin_assume_aligned(at, 4), sizeof(p));
    __builtin_memcpy(q, __builtin_assume_aligned(at + 3 * int64_t(R.W), 4), sizeof(q));
  } else {
    // 32-bit byte offsets from uniform row bases: 12 * 2^24 < 2^32
    const uint32_t off = uint32_t(fmaf(v0, float(R.W), u0)) * 12u;
    __builtin_memcpy(p, __builtin_assume_aligned(reinterpret_cast<const char*>(R.rays) + off, 4), sizeof(p));
    __builtin_memcpy(q, __builtin_assume_aligned(reinterpret_cast<const char*>(R.rays + 3 * R.W) + off, 4), sizeof(q));
  }
  C.u0 = u0;
  C.v0 = v0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    C.a[k] = target(k, p[k]);
    C.ab[k] = target(k, p[3 + k]) - C.a[k];
    C.c[k] = target(k, q[k]);
    C.cd[k] = target(k, q[3 + k]) - C.c[k];
  }
}

// A query's current point: the normal equations of the bilinear residual there, and its cost.
struct Normal {
  float a, b, dd, gu, gv;
};

// Bilinear sample of (ray image - target ray), i.e. the residual, at (fu, fv) in the cell; e: its change per unit of v.
template <bool BIG>
__device__ inline float cell_sample(const Cell<BIG>& C, float fu, float fv, float* s, float* e) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float top = fmaf(fu, C.ab[k], C.a[k]);
    const float bot = fmaf(fu, C.cd[k], C.c[k]);
    e[k] = bot - top;
    s[k] = fmaf(fv, e[k], top);
  }
  return fmaf(s[0], s[0], fmaf(s[1], s[1], s[2] * s[2]));
}

template <bool BIG>
__device__ inline Normal cell_normal(const Cell<BIG>& C, float fv, const float* s, const float* e) {
  float d[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) d[k] = fmaf(fv, C.cd[k] - C.ab[k], C.ab[k]);
  Normal N;
  N.a = fmaf(d[0], d[0], fmaf(d[1], d[1], d[2] * d[2]));
  N.b = fmaf(d[0], e[0], fmaf(d[1], e[1], d[2] * e[2]));
  N.dd = fmaf(e[0], e[0], fmaf(e[1], e[1], e[2] * e[2]));
  N.gu = fmaf(d[0], s[0], fmaf(d[1], s[1], d[2] * s[2]));
  N.gv = fmaf(e[0], s[0], fmaf(e[1], s[1], e[2] * s[2]));
  return N;
}

// One query at (u, v) of the reference to start with: returns idx (or -1), the final point and the trial steps.
template <bool BIG>
__device__ inline int32_t match_query(const RayImage& R, float4 x, float u, float v, const MatchConst& P, float* pu,
                                      float* pv, int* iters) {
  *pu = __builtin_nanf("");
  *pv = __builtin_nanf("");
  *iters = 0;
  const float dx2 = fmaf(x.x, x.x, fmaf(x.y, x.y, x.z * x.z));
  if (!finite3(x.x, x.y, x.z) || !(dx2 > 1e-18f)) return -1;
  const float dx = sqrtf(dx2);
  const float rdx = 1.0f / dx;
  const float X[3] = {x.x, x.y, x.z};
  const float t[3] = {x.x * rdx, x.y * rdx, x.z * rdx};
  const float u_max = float(R.W - 1), v_max = float(R.H - 1);
  Cell<BIG> C;
  // the first cell's differences take the target's product unrounded, later cells' the target ray
  fetch_cell(R, cell_origin<BIG>(u, R.W), cell_origin<BIG>(v, R.H), [&](int k, float p) { return fmaf(-X[k], rdx, p); }, C);
  float s[3], e[3];
  float c = cell_sample(C, u - float(C.u0), v - float(C.v0), s, e);
  if (isnan(c)) return -1;  // a hole
  Normal N = cell_normal(C, v - float(C.v0), s, e);  // unchanged by a rejected step, so rebuilt only on acceptance
  float lam = P.lambda0;
  int it = 0;
  bool hole = false;
#pragma unroll 1
  while (it < P.max_iters) {
    ++it;
    const float A = N.a * (1.0f + lam), D = N.dd * (1.0f + lam);
    const float det = fmaf(A, D, -(N.b * N.b));
    const bool det_ok = det > 0.0f;
    const float idet = __builtin_amdgcn_rcpf(det);  // hardware reciprocal (1 ulp)
    const float nu = fmaf(D, N.gu, -(N.b * N.gv)), nv = fmaf(A, N.gv, -(N.b * N.gu));
    // the median of three is the clamp (0 for a NaN)
    const float un = det_ok ? __builtin_amdgcn_fmed3f(fmaf(-nu, idet, u), 0.0f, u_max) : u;
    const float vn = det_ok ? __builtin_amdgcn_fmed3f(fmaf(-nv, idet, v), 0.0f, v_max) : v;
    const auto u0 = cell_origin<BIG>(un, R.W);
    const auto v0 = cell_origin<BIG>(vn, R.H);
    if (u0 != C.u0 || v0 != C.v0) fetch_cell(R, u0, v0, [&](int k, float p) { return p - t[k]; }, C);
    const float fv = vn - float(v0);
    const float cn = cell_sample(C, un - float(u0), fv, s, e);
    if (isnan(cn)) {
      hole = true;
      break;
    }
    const float step = fmaxf(fabsf(un - u), fabsf(vn - v));
    // A step that does not move (singular system, clamped or vanishing step) is rejected. Its cost is no test of that: c may
    // be of the first cell's differences and cn of a later fetch of the same cell, rounded otherwise and then below c.
    if (cn < c && (un != u || vn != v)) {
      u = un;
      v = vn;
      c = cn;
      lam = fmaxf(lam * 0.1f, P.lambda_min);
      N = cell_normal(C, fv, s, e);
    } else {
      lam *= 10.0f;
    }
    // A trial step shorter than the tolerance ends the search whether or not it is accepted (a
    // non-singular system: singular ones retry with a larger damping); the oracle takes the same rule.
    if (det_ok && step < P.step_tol) break;
  }
  *iters = it;
  if (hole) return -1;
  *pu = u;
  *pv = v;
  const float rr = sqrtf(c);
  if (!(rr <= P.ang_tol * sqrtf(fminf(N.a, N.dd)))) return -1;  // the smaller of |ds/du| and |ds/dv|
  const int mu = min(max(int(floorf(u + 0.5f)), 0), R.W - 1);
  const int mv = min(max(int(floorf(v + 0.5f)), 0), R.H - 1);
  const int32_t m = mv * R.W + mu;
  const float rm = R.range[m];
  if (!(rm > 0.f)) return -1;
  if (!(fabsf(dx - rm) <= P.range_tol * rm)) return -1;
  return m;
}

// Where a query's search starts: its own pixel, scaled to the reference's grid.
__device__ inline float start_scale(int n_ref, int n_qry) {
  return n_qry > 1 ? float(n_ref - 1) / float(n_qry - 1) : 0.0f;
}

__device__ inline float start_at(int q, float scale) {
#pragma clang fp contract(off)
  return float(q) * scale;  // rounded here
}

// One or two directions, one thread per query pixel: the tables are the kernel's arguments. One pair of 512 x 384 images
// (ray images, both directions, mutual check, gate): 57 us in seven launches and six table uploads, 27 us in four launches.
template <int DT, bool BIG>
__global__ __launch_bounds__(256) void k_match_few(MatchFew F, MatchConst P) {
  const bool second = blockIdx.x >= F.blocks0;  // uniform per block
  const MatchOne& D = F.d[second ? 1 : 0];
  const unsigned n = (blockIdx.x - (second ? F.blocks0 : 0u)) * 256u + threadIdx.x;
  if (n >= unsigned(D.Hq) * unsigned(D.Wq)) return;
  const RayImage R{D.rays, D.range, D.Hr, D.Wr};
  const float4 x = Px<DT>::load(D.qry, n);
  const int qv = int(n / unsigned(D.Wq)), qu = int(n - unsigned(qv) * unsigned(D.Wq));
  float pu, pv;
  int its;
  D.idx[n] = match_query<BIG>(R, x, start_at(qu, start_scale(D.Wr, D.Wq)), start_at(qv, start_scale(D.Hr, D.Hq)), P, &pu,
                              &pv, &its);
  if (D.p) {
    D.p[2 * int64_t(n)] = pu;
    D.p[2 * int64_t(n) + 1] = pv;
  }
  if (D.iters) D.iters[n] = its;
}

int launch_match_few(MatchFew F, int n_dirs, ds3_dtype dt, const MatchConst& P, hipStream_t s) {
  unsigned blocks[2] = {0, 0};
  bool big = false;
  for (int k = 0; k < n_dirs; ++k) {
    blocks[k] = unsigned((int64_t(F.d[k].Hq) * F.d[k].Wq + 255) / 256);
    big = big || match_big(F.d[k].Hr, F.d[k].Wr);
  }
  F.blocks0 = blocks[0];
  dim3 grid(blocks[0] + blocks[1]), block(256);
  if (grid.x == 0) return DS3_OK;
  if (dt == DS3_F32 && !big) hipLaunchKernelGGL((k_match_few<DS3_F32, false>), grid, block, 0, s, F, P);
  else if (dt == DS3_F32) hipLaunchKernelGGL((k_match_few<DS3_F32, true>), grid, block, 0, s, F, P);
  else if (!big) hipLaunchKernelGGL((k_match_few<DS3_BF16, false>), grid, block, 0, s, F, P);
  else hipLaunchKernelGGL((k_match_few<DS3_BF16, true>), grid, block, 0, s, F, P);
  return check_hip(hipGetLastError(), "k_match_few");
}

// The (entry, item) of block b; false for padding blocks. The bin's share of the items is a run of the entries' items
// laid end to end, so the last entry with prefix <= item is looked for, first where it is if all entries are alike.
__device__ inline bool locate_item(const ItemMap& M, int b, int& entry, int& item) {
  const int g = (b & 7) * M.per_bin + (b >> 3);
  if ((b >> 3) >= M.per_bin || g >= M.total) return false;
  int lo = 0, hi = M.n - 1;
  int mid = min(int(float(g) * (float(M.n) / float(M.total))), hi);
  while (lo < hi) {
    if (M.prefix[mid] > g) hi = mid - 1;
    else if (M.prefix[mid + 1] > g) lo = hi = mid;  // prefix has n + 1 entries
    else lo = mid + 1;
    mid = (lo + hi) >> 1;
  }
  entry = lo;
  item = g - M.prefix[lo];
  return true;
}

// Batched: a block is one wave and takes `per` strips of 16x4 query pixels of one direction, four strips to a 16x16 tile,
// one after the other; the next strip's queries are loaded before the current one's search. Blocks of one direction share
// an XCD, and directions with the same reference follow each other there. The LM trial-step count is
// summed per block and added to one of kStepStripes counters 128 B apart (block b to stripe b mod
// kStepStripes): a single counter hit by every wave becomes a hot spot of one L2 channel that stalls the
// whole launch.
// Bound by the gathers: a search is 5.5 cells in a chain, and the L1's return path is busy 87% of the time (35% waiting for
// the L2) at 6.6 waves per SIMD, with a vector instruction every 3.3 cycles; 9.3 GB from memory are no limit. 800 edges (276e6 queries) of a 200-keyframe graph: 4.1 ms with one tile per block of four waves (a search of
// the item map, the tables and the queries' latency per 64 queries), 16-byte rays and the references unsorted; 3.5 ms
// with four tiles per block and 12-byte rays; 3.35 ms with a wave per block. Tried without effect: the queries past the
// L2, the texels as 12 + 12 bytes (8 + 8 + 8: 3.7 ms).
template <int DT, bool BIG>
__global__ __launch_bounds__(64) void k_match_batched(const float* __restrict__ rays, const float* __restrict__ range,
                                                       const void* __restrict__ cross,
                                                       const MatchDir* __restrict__ dirs, ItemMap map, int per,
                                                       MatchConst P, int32_t* __restrict__ idx_tmp,
                                                       unsigned* __restrict__ step_stripes) {
  int entry, item;
  if (!locate_item(map, blockIdx.x, entry, item)) return;  // uniform per block
  const MatchDir D = dirs[entry];
  const RayImage R{rays + 3 * D.ref_off, range + D.ref_off, D.Hr, D.Wr};
  const float scale_u = start_scale(D.Wr, D.Wq), scale_v = start_scale(D.Hr, D.Hq);
  // a 16x16 tile of query pixels: their matches (and the LM steps towards them) cover a compact window of
  // the reference ray image, so the gathers share far more cache lines than a 256-pixel row segment's
  const int tiles_x = (D.Wq + kMatchTile - 1) / kMatchTile, tiles_y = (D.Hq + kMatchTile - 1) / kMatchTile;
  const int strips = kMatchStrips * tiles_x * tiles_y;
  int strip = item * per;
  const int last = min(strip + per, strips) - 1;
  int ty = strip / kMatchStrips / tiles_x, tx = strip / kMatchStrips - ty * tiles_x;
  const int lx = int(threadIdx.x % kMatchTile), ly = int(threadIdx.x / kMatchTile);
  int qu = tx * kMatchTile + lx, qv = ty * kMatchTile + strip % kMatchStrips * kStripRows + ly;
  int its = 0;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  if (qu < D.Wq && qv < D.Hq) x = Px<DT>::load(cross, D.qry_off + int64_t(qv) * D.Wq + qu);
#pragma unroll 1
  for (;; ++strip) {
    if (strip % kMatchStrips == kMatchStrips - 1 && ++tx == tiles_x) {
      tx = 0;
      ++ty;
    }
    const int qu_n = tx * kMatchTile + lx, qv_n = ty * kMatchTile + (strip + 1) % kMatchStrips * kStripRows + ly;
    float4 x_n = make_float4(0.f, 0.f, 0.f, 0.f);
    if (strip < last && qu_n < D.Wq && qv_n < D.Hq) x_n = Px<DT>::load(cross, D.qry_off + int64_t(qv_n) * D.Wq + qu_n);
    if (qu < D.Wq && qv < D.Hq) {
      float pu, pv;
      int n_it;
      idx_tmp[D.out_off + int64_t(qv) * D.Wq + qu] =
          match_query<BIG>(R, x, start_at(qu, scale_u), start_at(qv, scale_v), P, &pu, &pv, &n_it);
      its += n_it;
    }
    if (strip >= last) break;  // uniform per block
    x = x_n;
    qu = qu_n;
    qv = qv_n;
  }
  if (step_stripes) {
    its = wave_sum(its);
    if (threadIdx.x == 0 && its) atomicAdd(&step_stripes[(blockIdx.x % kStepStripes) * kStripeStride], unsigned(its));
  }
}

__global__ void k_sum_stripes(const unsigned* __restrict__ step_stripes, unsigned long long* __restrict__ out) {
  unsigned long long v = 0;
  for (int k = threadIdx.x; k < kStepStripes; k += blockDim.x) v += step_stripes[k * kStripeStride];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  __shared__ unsigned long long part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) *out = part[0] + part[1] + part[2] + part[3];
}

int launch_match_batched(const float* rays, const float* range, const void* cross, ds3_dtype dt, bool big,
                         const MatchDir* dirs, const ItemMap& map, int per, const MatchConst& P, int32_t* idx_tmp,
                         unsigned* step_stripes, hipStream_t s) {
  dim3 grid(8 * map.per_bin), block(64);
  if (grid.x == 0) return DS3_OK;
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, rays, range, cross, dirs, map, per, P, idx_tmp, step_stripes);
  };
  if (dt == DS3_F32 && !big) run(k_match_batched<DS3_F32, false>);
  else if (dt == DS3_F32) run(k_match_batched<DS3_F32, true>);
  else if (!big) run(k_match_batched<DS3_BF16, false>);
  else run(k_match_batched<DS3_BF16, true>);
  return check_hip(hipGetLastError(), "k_match_batched");
}

int launch_sum_stripes(const unsigned* step_stripes, unsigned long long* out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_stripes, dim3(1), dim3(256), 0, s, step_stripes, out);
  return check_hip(hipGetLastError(), "k_sum_stripes");
}

// --------------------------------------------------------------------------------------------------
// Mutual check + nu counts. Side J (pixels of j): final idx and valid mask; side I (pixels of i):
// count only. Every block writes its tile's count to its own slot of the partials (no atomics: the
// blocks of one side would otherwise all hit one counter), then k_nu sums each side in a fixed order.
// --------------------------------------------------------------------------------------------------
// One block: `per` runs of kMutualPx pixels, one after the other; the next run's forward matches and confidences are loaded
// before the current one's gathers. Bound by memory: 4.3 GB (the L1 waits for the L2 68% of the time) at 5.0 TB/s, as a large
// copy; both sides of an edge run on one XCD and share its L2. 276e6 pixels of 800 edges: 1.07 ms with one run per block
// (the map's lookup, the tables and the first loads are a chain of their own), 0.86 ms with eight; 0.71 ms without the
// confidences.
__device__ inline void mutual_tiles_of(const MutualDir& M, int item, int per, const MatchConst& P,
                                       const int32_t* __restrict__ idx_tmp, int32_t* __restrict__ idx_final,
                                       uint8_t* __restrict__ valid, unsigned* __restrict__ part) {
  constexpr int kPer = kMutualPx / 256;
  const int n_self = M.H_self * M.W_self, n_other = M.H_other * M.W_other;  // at most INT32_MAX
  const int32_t* fwd = idx_tmp + M.fwd_off;
  const int32_t* bwd = idx_tmp + M.bwd_off;
  const unsigned w = unsigned(M.W_self);
  const int64_t first = int64_t(item) * per * kMutualPx + threadIdx.x;
  int32_t m_next[kPer];
  float cs_next[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int64_t n = first + u * 256;
    m_next[u] = n < n_self ? fwd[n] : -1;
    cs_next[u] = n < n_self ? M.conf_self[n] : 0.0f;
  }
  int hit = 0;
#pragma unroll 1
  for (int r = 0; r < per; ++r) {
    // four independent pixels per thread, every load of a stage issued before its first use:
    // the backward matches and the other's confidences, then the next run
    int32_t m[kPer], n2[kPer];
    float cs[kPer], co[kPer];
    const int64_t at = first + int64_t(r) * kMutualPx;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      m[u] = m_next[u] < n_other ? m_next[u] : -1;
      cs[u] = cs_next[u];
      n2[u] = m[u] >= 0 ? bwd[m[u]] : -1;
      co[u] = m[u] >= 0 ? M.conf_other[m[u]] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int64_t n = at + kMutualPx + u * 256;
      const bool more = r + 1 < per && n < n_self;
      m_next[u] = more ? fwd[n] : -1;
      cs_next[u] = more ? M.conf_self[n] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int64_t n = at + u * 256;
      if (n >= n_self) continue;
      bool ok = m[u] >= 0 && n2[u] >= 0 && n2[u] < n_self;
      if (ok) {
        const unsigned p = unsigned(n2[u]), q = unsigned(n);
        const unsigned py = p / w, qy = q / w;
        const int du = abs(int(p - py * w) - int(q - qy * w));
        const int dv = abs(int(py) - int(qy));
        ok = max(du, dv) <= P.radius;
      }
      if (ok) hit += (sqrt(double(co[u]) * double(cs[u])) >= P.q_min) ? 1 : 0;
      if (M.write_out) {
        idx_final[M.out_off + n] = ok ? m[u] : -1;
        valid[M.out_off + n] = ok ? 1 : 0;
      }
    }
  }
  hit = wave_sum(hit);
  __shared__ int s[4];
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = hit;
  __syncthreads();
  if (threadIdx.x == 0) part[M.part_off + item] = unsigned(s[0] + s[1] + s[2] + s[3]);
}

__global__ __launch_bounds__(256) void k_mutual(const MutualDir* __restrict__ md, ItemMap map, int per, MatchConst P,
                                                const int32_t* __restrict__ idx_tmp, int32_t* __restrict__ idx_final,
                                                uint8_t* __restrict__ valid, unsigned* __restrict__ part) {
  int entry, item;
  if (!locate_item(map, blockIdx.x, entry, item)) return;  // uniform per block
  const MutualDir M = md[entry];
  mutual_tiles_of(M, item, per, P, idx_tmp, idx_final, valid, part);
}

int launch_mutual(const MutualDir* md, const ItemMap& map, int per, const MatchConst& P, const int32_t* idx_tmp,
                  int32_t* idx_final, uint8_t* valid, unsigned* part, hipStream_t s) {
  if (map.per_bin <= 0) return DS3_OK;
  hipLaunchKernelGGL(k_mutual, dim3(8 * map.per_bin), dim3(256), 0, s, md, map, per, P, idx_tmp, idx_final, valid, part);
  return check_hip(hipGetLastError(), "k_mutual");
}

// The two sides of one edge.
__global__ __launch_bounds__(256) void k_mutual_pair(MutualPair M, MatchConst P, const int32_t* __restrict__ idx_tmp,
                                                     int32_t* __restrict__ idx_final, uint8_t* __restrict__ valid,
                                                     unsigned* __restrict__ part) {
  const bool second = int(blockIdx.x) >= M.tiles0;
  mutual_tiles_of(M.d[second ? 1 : 0], int(blockIdx.x) - (second ? M.tiles0 : 0), 1, P, idx_tmp, idx_final, valid, part);
}

int launch_mutual_pair(const MutualPair& M, int tiles, const MatchConst& P, const int32_t* idx_tmp, int32_t* idx_final,
                       uint8_t* valid, unsigned* part, hipStream_t s) {
  if (tiles <= 0) return DS3_OK;
  hipLaunchKernelGGL(k_mutual_pair, dim3(tiles), dim3(256), 0, s, M, P, idx_tmp, idx_final, valid, part);
  return check_hip(hipGetLastError(), "k_mutual_pair");
}

// One wave per side: lanes stride the side's tile partials, then a fixed-shape wave sum. nu = count / pixels in double;
// admit = min(nu_i, nu_j) >= nu_min (same arithmetic as a double sum).
__device__ inline void nu_edge(const NuSide& S, int side, int e, bool live, const unsigned* __restrict__ part,
                               double nu_min, float* __restrict__ nu, int32_t* __restrict__ admit, double (*share)[2]) {
  const int lane = threadIdx.x & 63;
  unsigned v = 0;
  if (live)
    for (int k = lane; k < S.n_parts; k += 64) v += part[S.first + k];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  const int row = threadIdx.x >> 7;
  if (lane == 0) share[row][side] = live ? double(v) / double(S.npx) : 0.0;
  __syncthreads();
  if (!live || side != 0 || lane != 0) return;
  const double ni = share[row][0], nj = share[row][1];
  if (nu) {
    nu[2 * e] = float(ni);
    nu[2 * e + 1] = float(nj);
  }
  if (admit) admit[e] = (fmin(ni, nj) >= nu_min) ? 1 : 0;
}

__global__ __launch_bounds__(256) void k_nu(const unsigned* __restrict__ part, const NuSide* __restrict__ sides,
                                            int n_edges, double nu_min, float* __restrict__ nu,
                                            int32_t* __restrict__ admit) {
  __shared__ double share[2][2];
  const int slot = blockIdx.x * 4 + int(threadIdx.x >> 6), e = slot >> 1;
  const bool live = e < n_edges;
  nu_edge(live ? sides[slot] : NuSide{}, slot & 1, e, live, part, nu_min, nu, admit, share);
}

int launch_nu(const unsigned* part, const NuSide* sides, int n_edges, double nu_min, float* nu, int32_t* admit,
              hipStream_t s) {
  if (n_edges <= 0) return DS3_OK;
  hipLaunchKernelGGL(k_nu, dim3((n_edges + 1) / 2), dim3(256), 0, s, part, sides, n_edges, nu_min, nu, admit);
  return check_hip(hipGetLastError(), "k_nu");
}

__global__ __launch_bounds__(128) void k_nu_pair(const unsigned* __restrict__ part, NuSide i, NuSide j, double nu_min,
                                                 float* __restrict__ nu, int32_t* __restrict__ admit) {
  __shared__ double share[2][2];
  const int side = threadIdx.x >> 6;
  nu_edge(side ? j : i, side, 0, true, part, nu_min, nu, admit, share);
}

int launch_nu_pair(const unsigned* part, const NuSide& i, const NuSide& j, double nu_min, float* nu, int32_t* admit,
                   hipStream_t s) {
  hipLaunchKernelGGL(k_nu_pair, dim3(1), dim3(128), 0, s, part, i, j, nu_min, nu, admit);
  return check_hip(hipGetLastError(), "k_nu_pair");
}

}  // namespace ds3
