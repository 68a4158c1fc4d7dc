// Terminal segment-level depth refinement (Sec. III-E, eqs. (8)-(10)).
//
// Segmentation (once per plan): per keyframe, SLIC over canonical surface normals and normalised
// log-range, pixels with confidence below C_min excluded, segments with fewer than min_seg_px valid pixels
// excluded. Features are computed in float64 in a fixed operation order and quantised to integers, and the
// clustering runs in exact int64 arithmetic, so the labels do not depend on summation order:
//   F = (round(Q (n + 1)) x3, round(Q l)), Q = 1024; S = round(sqrt(HW / M_k)); one centre per grid cell;
//   D = S^2 |F_p - F_c|^2 + 512^2 |xy_p - xy_c|^2 over the centres of the 3x3 cells around the pixel's cell
//   (ties: lowest centre index); centres move to the floor of their members' mean; fixed iteration count.
// Centre updates are integer sums, so the order in which the assignment's blocks add their members does not matter.
// Boundary table: for 4-adjacent pixels of two valid segments g != h of a keyframe, the log-range difference
// ln|X(p)| - ln|X(p')| (p in g) is summed into slot (g -> h) and its negative into (h -> g); h's grid cell is
// within 3 cells of g's, so each segment keeps 7 x 7 slots indexed by the cell offset. Sums are int64 fixed
// point (2^-40), so the table is independent of the order of the atomic adds.
//
// One refinement iteration (Jacobi-style damped Newton, eqs. 8-10):
//   data: for every match (m, n) of edge (i, j), X_j(eta) = X_j exp(eta_h), X_i(eta) = X_i exp(eta_g),
//     r = sqrt(q)/sigma_point (T_ij X_j(eta) - X_i(eta)), Huber weights w; the segments' diagonal
//     H += w |J|^2 and gradient g += w J.r with J_h = sqrt(q)/sigma (sR_ij X_j(eta)), J_g = -sqrt(q)/sigma
//     X_i(eta) -- one block per (edge, 4096-pixel tile of j) accumulates into LDS tables indexed by the
//     segment's slot in its keyframe (at most 256 per keyframe) and flushes them with float64 atomics;
//   step: per segment, boundary (lambda_smooth per pair, lambda_smooth r_b in the gradient) and prior
//     (lambda_prior, lambda_prior eta) terms, delta = clip(-g / ((1 + lambda_lm) H), +-eta_max), anchor
//     keyframes' segments fixed; eta is double-buffered so every segment reads the iteration's input.
// The objective reported per iteration is E' = sum rho + (lambda_smooth/2) sum_B r_b^2 +
// (lambda_prior/2) sum eta^2 at the iteration's input eta.
#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "common.hpp"
#include "internal.hpp"
#include "sim3.hpp"

namespace ds3 {

constexpr int kMaxSegPerKf = 256;  // LDS tables of the data kernel are indexed by a keyframe's segment slot
constexpr int kSlots = 49;         // 7 x 7 grid-cell offsets of a boundary neighbour
constexpr double kFix = 1099511627776.0;  // 2^40, fixed-point scale of the boundary sums
constexpr int kDepthThreads = 256;

struct DepthKf {
  int64_t off;      // arena pixel offset
  int32_t H, W, S, nx, ny;
  int32_t seg_base;  // first global segment id
  int32_t anchor;
  int32_t pad;
};

struct DepthConst {
  double conf_min;
  float inv_sigma, kappa;
  double lambda_smooth, lambda_prior, lambda_lm, eta_max;
};

// ---- features --------------------------------------------------------------------------------------
template <int DT>
__device__ inline void load_xyz(const void* arena, int64_t px, double* X, double& C) {
  const float4 v = Px<DT>::load(arena, px);
  X[0] = v.x;
  X[1] = v.y;
  X[2] = v.z;
  C = v.w;
}

// A hole: a non-finite component or |X| <= 1e-9 (products and sums in the order of the reference: (x x + y y) + z z). In
// float32 but for a largest component of up to 2e-9, where float64 decides.
__device__ inline bool is_hole(const float4& v) {
  if (fmaf(v.x, 0.0f, fmaf(v.y, 0.0f, v.z * 0.0f)) != 0.0f) return true;  // NaN with a NaN or an infinity
  if (fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fabsf(v.z)) > 2e-9f) return false;
  // |X| > 1e-9 without the square root: the largest double whose (correctly rounded) root is at most 1e-9
  constexpr double kHole2 = 0x1.2725dd1d243adp-60;
  const double x = v.x, y = v.y, z = v.z;
  return !((x * x + y * y) + z * z > kHole2);
}

__device__ inline double log_range(const double* X) {
  const double a = isfinite(X[0]) ? X[0] : 0.0, b = isfinite(X[1]) ? X[1] : 0.0, c = isfinite(X[2]) ? X[2] : 0.0;
  const double n = sqrt((a * a + b * b) + c * c);
  return log(fmax(n, 1e-300));
}

// Per keyframe: min and max of ln|X| over its valid pixels, in kRangeParts blocks (one block per keyframe leaves most of
// the chip idle: 610 us for 200 keyframes, 163 us with 16, 94 us with the extremes taken of |X|^2 and one logarithm
// each at the end). The extremes of the parts are exact whatever their order.
constexpr int kRangeParts = 16;

template <int DT>
__global__ __launch_bounds__(kDepthThreads) void k_dr_logrange(const void* __restrict__ arena,
                                                               const DepthKf* __restrict__ kfs, DepthConst dc,
                                                               double* __restrict__ lmin, double* __restrict__ lmax) {
  const DepthKf K = kfs[blockIdx.y];
  const int n = K.H * K.W;
  double lo = INFINITY, hi = -INFINITY;
  for (int64_t p = blockIdx.x * kDepthThreads + threadIdx.x; p < n; p += kRangeParts * kDepthThreads) {
    const float4 v = Px<DT>::load(arena, K.off + p);
    if (is_hole(v) || !(double(v.w) >= dc.conf_min)) continue;
    const double x = v.x, y = v.y, z = v.z;
    const double n2 = (x * x + y * y) + z * z;
    lo = fmin(lo, n2);
    hi = fmax(hi, n2);
  }
  // no pixel: they stay infinite
  lo = log(sqrt(lo));
  hi = hi > 0.0 ? log(sqrt(hi)) : hi;
  __shared__ double slo[kDepthThreads / kWave], shi[kDepthThreads / kWave];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, kWave));
    hi = fmax(hi, __shfl_xor(hi, off, kWave));
  }
  if ((threadIdx.x & (kWave - 1)) == 0) {
    slo[threadIdx.x / kWave] = lo;
    shi[threadIdx.x / kWave] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kDepthThreads / kWave; ++w) {
      lo = fmin(lo, slo[w]);
      hi = fmax(hi, shi[w]);
    }
    lmin[blockIdx.y * kRangeParts + blockIdx.x] = lo;
    lmax[blockIdx.y * kRangeParts + blockIdx.x] = hi;
  }
}

// Correctly rounded a / d from r = recip_f64(d): two Newton-Raphson steps on the estimate of 1 / d, then Markstein's
// correction of the quotient by its residual (a division without its scaling: for d, and any a with |a| <= |d|, far from the
// ends of the range; a quotient that underflows may lose its last bits).
__device__ inline double recip_f64(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = fma(y, fma(-d, y, 1.0), y);
  return fma(y, fma(-d, y, 1.0), y);
}
__device__ inline double div_f64(double a, double d, double r) {
  const double q = a * r;
  return fma(fma(-q, d, a), r, q);
}
__device__ inline bool div_safe(double d) { return d > 1e-100 && d < 1e100; }

// The extremes of keyframe k's parts: {least, greatest - least, 1 / that (0 when a division has to do)}.
__global__ void k_dr_range(int n_kf, const double* __restrict__ lmin, const double* __restrict__ lmax,
                           double* __restrict__ range) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_kf) return;
  double lo = INFINITY, hi = -INFINITY;
#pragma unroll
  for (int q = 0; q < kRangeParts; ++q) {
    lo = fmin(lo, lmin[k * kRangeParts + q]);
    hi = fmax(hi, lmax[k * kRangeParts + q]);
  }
  const double d = hi > lo ? hi - lo : 0.0;
  range[3 * k] = lo;
  range[3 * k + 1] = d;
  range[3 * k + 2] = div_safe(d) ? recip_f64(d) : 0.0;
}

// Quantised features of every pixel of keyframe blockIdx.y (4 x uint16, packed; all zero for an invalid pixel and for no
// other: a valid one with n_x = -1 has n_y = n_z = 0, which quantise to 1024). Normal: cross product of central differences (one-sided at the
// border), unit length, oriented towards the camera; zero where a pixel used is a hole. Bound by float64 operations at half
// the rate: with the extremes of the 16 parts taken by every pixel and a division per component it took 474 us for 200
// keyframes of 512 x 384, now 379 us.
template <int DT>
__global__ __launch_bounds__(kDepthThreads) void k_dr_features(const void* __restrict__ arena,
                                                               const DepthKf* __restrict__ kfs, DepthConst dc,
                                                               const double* __restrict__ range,
                                                               uint2* __restrict__ feat) {
  const DepthKf K = kfs[blockIdx.y];
  const int p = blockIdx.x * kDepthThreads + threadIdx.x;
  if (p >= K.H * K.W) return;
  const int v = p / K.W, u = p - v * K.W;
  const float4 P = Px<DT>::load(arena, K.off + p);
  const double X[3] = {P.x, P.y, P.z};
  const bool valid = !is_hole(P) && double(P.w) >= dc.conf_min;
  const int64_t gp = K.off + p;
  if (!valid) {
    feat[gp] = make_uint2(0u, 0u);
    return;
  }
  auto nb = [&](int uu, int vv, double* Y) {
    const float4 Q = Px<DT>::load(arena, K.off + int64_t(vv) * K.W + uu);
    const bool h = is_hole(Q);
    Y[0] = h ? 0.0f : Q.x;
    Y[1] = h ? 0.0f : Q.y;
    Y[2] = h ? 0.0f : Q.z;
    return h;
  };
  double A[3], B[3], Cc[3], Dd[3];
  const int u0 = max(u - 1, 0), u1 = min(u + 1, K.W - 1), v0 = max(v - 1, 0), v1 = min(v + 1, K.H - 1);
  bool bad = nb(u1, v, A);
  bad |= nb(u0, v, B);
  bad |= nb(u, v1, Cc);
  bad |= nb(u, v0, Dd);
  const double du[3] = {A[0] - B[0], A[1] - B[1], A[2] - B[2]};
  const double dv[3] = {Cc[0] - Dd[0], Cc[1] - Dd[1], Cc[2] - Dd[2]};
  double c[3] = {du[1] * dv[2] - du[2] * dv[1], du[2] * dv[0] - du[0] * dv[2], du[0] * dv[1] - du[1] * dv[0]};
  const double ln = sqrt((c[0] * c[0] + c[1] * c[1]) + c[2] * c[2]);
  double n[3] = {0.0, 0.0, 0.0};
  if (!bad && ln > 0.0 && isfinite(ln)) {
    if (div_safe(ln)) {
      const double r = recip_f64(ln);
#pragma unroll
      for (int q = 0; q < 3; ++q) n[q] = div_f64(c[q], ln, r);
    } else {
      n[0] = c[0] / ln;
      n[1] = c[1] / ln;
      n[2] = c[2] / ln;
    }
  }
  if ((n[0] * X[0] + n[1] * X[1]) + n[2] * X[2] > 0.0) {
    n[0] = -n[0];
    n[1] = -n[1];
    n[2] = -n[2];
  }
  const double lo = range[3 * blockIdx.y], span = range[3 * blockIdx.y + 1], inv = range[3 * blockIdx.y + 2];
  const double above = log(sqrt((X[0] * X[0] + X[1] * X[1]) + X[2] * X[2])) - lo;
  const double ell = span > 0.0 ? (inv > 0.0 ? div_f64(above, span, inv) : above / span) : 0.0;
  const uint32_t f0 = uint32_t(floor(1024.0 * (n[0] + 1.0) + 0.5));
  const uint32_t f1 = uint32_t(floor(1024.0 * (n[1] + 1.0) + 0.5));
  const uint32_t f2 = uint32_t(floor(1024.0 * (n[2] + 1.0) + 0.5));
  const uint32_t f3 = uint32_t(floor(1024.0 * ell + 0.5));
  feat[gp] = make_uint2(f0 | (f1 << 16), f2 | (f3 << 16));
}

__device__ inline void unpack_feat(uint2 w, int64_t* F) {
  F[0] = int64_t(w.x & 0xffffu);
  F[1] = int64_t(w.x >> 16);
  F[2] = int64_t(w.y & 0xffffu);
  F[3] = int64_t(w.y >> 16);
}

// ---- SLIC --------------------------------------------------------------------------------------------
// Centre c of keyframe k: cen[6 (seg_base + c) + {x, y, F0..F3}] (int64).
__global__ void k_slic_init(const DepthKf* __restrict__ kfs, int n_kf, const uint2* __restrict__ feat,
                            int64_t* __restrict__ cen) {
  const int k = blockIdx.y;
  if (k >= n_kf) return;
  const DepthKf K = kfs[k];
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= K.nx * K.ny) return;
  const int cy = c / K.nx, cx = c - cy * K.nx;
  const int px = min(cx * K.S + K.S / 2, K.W - 1), py = min(cy * K.S + K.S / 2, K.H - 1);
  int64_t F[4];
  unpack_feat(feat[K.off + int64_t(py) * K.W + px], F);
  int64_t* o = cen + 6 * int64_t(K.seg_base + c);
  o[0] = px;
  o[1] = py;
  for (int q = 0; q < 4; ++q) o[2 + q] = F[q];
}

// One iteration's assignment and sums: each valid pixel takes the nearest of the centres of the 3x3 grid cells around
// its own and adds (1, x, y, F) to that centre's sums. A block takes 64 x 32 pixels, a thread eight rows of one column;
// the keyframe's centres (at most 256) sit in LDS, and a candidate is read once for all rows that see it. Sums first run
// over a thread's consecutive rows of one label, then over the block in LDS (three 64-bit adds per run: count, x and y
// relative to the tile packed with 16, 24 and 24 bits, the features two to a word), and each centre the block touched is
// flushed with seven global adds. All integer, so the result does not depend on the order.
// Bound by the vector units (about 13 instructions per pixel and candidate: packed 16-bit feature differences, their
// squares by 16-bit dot products, one 64-bit product) with 8 B read per pixel: 0.50 + 0.48 ms per iteration for 34.4 M
// pixels as an assignment with 64-bit arithmetic throughout and a gather of each centre's members over 3x3 cells,
// 0.15 ms now. The labels are written by the last iteration only.
// WIDE: an image side above 32767, where squared pixel offsets need 64 bits.
constexpr int kSlicTW = 64, kSlicTH = 32, kSlicRows = 8;

typedef short s16x2 __attribute__((ext_vector_type(2)));

__device__ inline uint32_t feat_dist2(uint2 a, uint2 b) {
  const s16x2 e0 = __builtin_bit_cast(s16x2, a.x) - __builtin_bit_cast(s16x2, b.x);
  const s16x2 e1 = __builtin_bit_cast(s16x2, a.y) - __builtin_bit_cast(s16x2, b.y);
  return uint32_t(__builtin_amdgcn_sdot2(e0, e0, __builtin_amdgcn_sdot2(e1, e1, 0, false), false));
}

template <bool WIDE>
__global__ __launch_bounds__(kDepthThreads) void k_slic_pass(const DepthKf* __restrict__ kfs,
                                                             const uint2* __restrict__ feat,
                                                             const int64_t* __restrict__ cen,
                                                             unsigned long long* __restrict__ sums,
                                                             int32_t* __restrict__ label, int last) {
  static_assert(kSlicTW == kWave && kSlicTH == kSlicRows * (kDepthThreads / kWave), "one wave per eight rows");
  __shared__ int2 sp[kMaxSegPerKf];   // centre positions
  __shared__ uint2 sf[kMaxSegPerKf];  // centre features, packed as the pixels'
  __shared__ unsigned long long acc[3][kMaxSegPerKf];
  const DepthKf K = kfs[blockIdx.y];
  const int tiles_x = (K.W + kSlicTW - 1) / kSlicTW;
  const int ty = int(blockIdx.x) / tiles_x;
  const int x0 = (int(blockIdx.x) - ty * tiles_x) * kSlicTW, y0 = ty * kSlicTH;
  if (y0 >= K.H) return;  // uniform per block
  const int M = K.nx * K.ny;
  for (int c = threadIdx.x; c < M; c += kDepthThreads) {
    const int64_t* o = cen + 6 * int64_t(K.seg_base + c);
    sp[c] = make_int2(int(o[0]), int(o[1]));
    sf[c] = make_uint2(uint32_t(o[2]) | (uint32_t(o[3]) << 16), uint32_t(o[4]) | (uint32_t(o[5]) << 16));
    acc[0][c] = acc[1][c] = acc[2][c] = 0;
  }
  const int x = x0 + int(threadIdx.x & (kWave - 1));
  const int yb = y0 + __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave) * kSlicRows;  // first row of the wave
  uint2 F[kSlicRows];
#pragma unroll
  for (int r = 0; r < kSlicRows; ++r)
    F[r] = (x < K.W && yb + r < K.H) ? feat[K.off + int64_t(yb + r) * K.W + x] : make_uint2(0u, 0u);
  __syncthreads();
  if (x < K.W && yb < K.H) {
    uint64_t best[kSlicRows];
    int lab[kSlicRows], gy[kSlicRows];
    const int gx = min(x / K.S, K.nx - 1);
    int row = yb / K.S;
#pragma unroll
    for (int r = 0; r < kSlicRows; ++r) {
      best[r] = ~0ull;
      lab[r] = -1;
      while (yb + r >= (row + 1) * K.S) ++row;
      gy[r] = min(row, K.ny - 1);
    }
    const uint32_t S2 = uint32_t(K.S) * uint32_t(K.S);
    const int cx0 = max(gx - 1, 0), cx1 = min(gx + 1, K.nx - 1);
    const int cy1 = min(gy[kSlicRows - 1] + 1, K.ny - 1);
    for (int cy = max(gy[0] - 1, 0); cy <= cy1; ++cy)  // increasing centre index: ties go to the lowest
      for (int cx = cx0; cx <= cx1; ++cx) {
        const int c = cy * K.nx + cx;
        const int2 P = sp[c];
        const uint2 G = sf[c];
        const int ex = x - P.x;
#pragma unroll
        for (int r = 0; r < kSlicRows; ++r) {
          if (abs(cy - gy[r]) > 1) continue;  // uniform per wave
          const int ey = yb + r - P.y;
          uint64_t d;
          if constexpr (WIDE) {
            d = uint64_t(int64_t(ex) * ex + int64_t(ey) * ey) << 18;
          } else {
            d = uint64_t(uint32_t(__mul24(ex, ex) + __mul24(ey, ey))) << 18;
          }
          d += uint64_t(S2) * feat_dist2(F[r], G);
          if (d < best[r]) {
            best[r] = d;
            lab[r] = c;
          }
        }
      }
    int cur = -1;
    unsigned long long a0 = 0, a1 = 0, a2 = 0;
#pragma unroll
    for (int r = 0; r < kSlicRows; ++r) {
      if (yb + r >= K.H) break;
      const bool valid = (F[r].x | F[r].y) != 0u;
      if (last) label[K.off + int64_t(yb + r) * K.W + x] = valid ? lab[r] : -1;
      if (!valid) continue;
      if (lab[r] != cur) {
        if (cur >= 0) {
          atomicAdd(&acc[0][cur], a0);
          atomicAdd(&acc[1][cur], a1);
          atomicAdd(&acc[2][cur], a2);
        }
        cur = lab[r];
        a0 = a1 = a2 = 0;
      }
      a0 += 1ull | (uint64_t(uint32_t(x - x0)) << 16) | (uint64_t(uint32_t(yb + r - y0)) << 40);
      a1 += uint64_t(F[r].x & 0xffffu) | (uint64_t(F[r].x >> 16) << 32);
      a2 += uint64_t(F[r].y & 0xffffu) | (uint64_t(F[r].y >> 16) << 32);
    }
    if (cur >= 0) {
      atomicAdd(&acc[0][cur], a0);
      atomicAdd(&acc[1][cur], a1);
      atomicAdd(&acc[2][cur], a2);
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < M; c += kDepthThreads) {
    const unsigned long long v0 = acc[0][c], v1 = acc[1][c], v2 = acc[2][c];
    const unsigned long long n = v0 & 0xffffu;
    if (n == 0) continue;
    unsigned long long* o = sums + 7 * int64_t(K.seg_base + c);
    atomicAdd(o, n);
    atomicAdd(o + 1, ((v0 >> 16) & 0xffffffu) + n * uint64_t(x0));
    atomicAdd(o + 2, (v0 >> 40) + n * uint64_t(y0));
    atomicAdd(o + 3, v1 & 0xffffffffu);
    atomicAdd(o + 4, v1 >> 32);
    atomicAdd(o + 5, v2 & 0xffffffffu);
    atomicAdd(o + 6, v2 >> 32);
  }
}

// Each centre moves to the floor of its members' mean (no members: unchanged); writes the member count and clears the
// sums for the next iteration.
__global__ __launch_bounds__(kDepthThreads) void k_slic_move(unsigned long long* __restrict__ sums, int n_seg,
                                                             int64_t* __restrict__ cen, int32_t* __restrict__ cnt) {
  const int s = blockIdx.x * kDepthThreads + threadIdx.x;
  if (s >= n_seg) return;
  unsigned long long* o = sums + 7 * int64_t(s);
  const unsigned long long n = o[0];
  if (n > 0)
    for (int k = 0; k < 6; ++k) cen[6 * int64_t(s) + k] = int64_t(o[1 + k] / n);
  cnt[s] = int32_t(n);
  for (int k = 0; k < 7; ++k) o[k] = 0;
}

// Final labels: global segment id, or -1 for invalid pixels and for segments with fewer than min_px pixels; and the
// same as 16-bit slots of the keyframe (kNoSlot for -1), which the data kernel gathers.
constexpr uint32_t kNoSlot = 0xffffu;

__global__ __launch_bounds__(kDepthThreads) void k_label_finalize(const DepthKf* __restrict__ kfs,
                                                                  const int32_t* __restrict__ cnt, int min_px,
                                                                  int32_t* __restrict__ label,
                                                                  uint16_t* __restrict__ slot,
                                                                  uint8_t* __restrict__ seg_valid) {
  const DepthKf K = kfs[blockIdx.y];
  const int p = blockIdx.x * kDepthThreads + threadIdx.x;
  if (p < K.nx * K.ny) seg_valid[K.seg_base + p] = cnt[K.seg_base + p] >= min_px ? 1 : 0;
  if (p >= K.H * K.W) return;
  const int64_t gp = K.off + p;
  const int l = label[gp];
  const bool keep = l >= 0 && cnt[K.seg_base + l] >= min_px;
  if (l >= 0) label[gp] = keep ? K.seg_base + l : -1;
  slot[gp] = uint16_t(keep ? uint32_t(l) : kNoSlot);
}

// ---- boundary table -------------------------------------------------------------------------------------
__device__ inline int slot_of(const DepthKf& K, int g_local, int h_local) {
  const int gy = g_local / K.nx, gx = g_local - gy * K.nx;
  const int hy = h_local / K.nx, hx = h_local - hy * K.nx;
  return (hy - gy + 3) * 7 + (hx - gx + 3);
}

// Boundary pairs are few (about 8% of the pixels with segments 31 pixels wide), so a block first collects those of its
// 64 x 32 pixels from the labels alone into a list in LDS (entry: pixel of the tile, direction), then its threads take
// the list's entries side by side: both logarithms, and the pair's difference added to a hash table in LDS keyed by (the
// lower segment, its slot of the other). One entry per distinct pair is flushed to both orientations. 2.0 ms for 34.4 M
// pixels with a logarithm at every pixel and four device-scope atomics per boundary pair; 0.23 ms now. A pair that finds
// no room in the table goes to memory directly.
constexpr int kPairHash = 512;  // entries; a tile of 31-pixel segments holds about 40 distinct pairs
constexpr int kPairProbes = 16;

__device__ inline void add_pair(unsigned long long* __restrict__ bsum, int32_t* __restrict__ bcnt, const DepthKf& K,
                                int gl, int hl, unsigned long long q, int n) {
  const int64_t a = int64_t(K.seg_base + gl) * kSlots + slot_of(K, gl, hl);
  const int64_t b = int64_t(K.seg_base + hl) * kSlots + slot_of(K, hl, gl);
  atomicAdd(&bsum[a], q);
  atomicAdd(&bcnt[a], n);
  atomicAdd(&bsum[b], 0ull - q);
  atomicAdd(&bcnt[b], n);
}

template <int DT>
__global__ __launch_bounds__(kDepthThreads) void k_dr_boundary(const void* __restrict__ arena,
                                                               const DepthKf* __restrict__ kfs,
                                                               const int32_t* __restrict__ label,
                                                               unsigned long long* __restrict__ bsum,
                                                               int32_t* __restrict__ bcnt) {
  __shared__ uint16_t list[2 * kSlicTW * kSlicTH];
  __shared__ int n_list;
  __shared__ int key[kPairHash], cnt[kPairHash];
  __shared__ unsigned long long sum[kPairHash];
  const DepthKf K = kfs[blockIdx.y];
  const int tiles_x = (K.W + kSlicTW - 1) / kSlicTW;
  const int ty = int(blockIdx.x) / tiles_x;
  const int x0 = (int(blockIdx.x) - ty * tiles_x) * kSlicTW, y0 = ty * kSlicTH;
  if (y0 >= K.H) return;  // uniform per block
  if (threadIdx.x == 0) n_list = 0;
  for (int q = threadIdx.x; q < kPairHash; q += kDepthThreads) {
    key[q] = -1;
    cnt[q] = 0;
    sum[q] = 0;
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int yw = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave) * kSlicRows;  // first row of the wave
  const int x = x0 + lane;
  const bool in_x = x < K.W, right_x = x + 1 < K.W;
  const int32_t* __restrict__ lab = label + K.off;
  // the wave's rows, the row below and each row's right neighbours, all loads first
  int g[kSlicRows + 1], rt[kSlicRows];
#pragma unroll
  for (int r = 0; r <= kSlicRows; ++r) {
    const int y = y0 + yw + r;
    const int64_t at = int64_t(y) * K.W + x;
    g[r] = (in_x && y < K.H) ? lab[at] : -1;
    if (r < kSlicRows) rt[r] = (right_x && y < K.H) ? lab[at + 1] : -1;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSlicRows; ++r)
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      const int h = dir == 0 ? rt[r] : g[r + 1];
      const bool pair = g[r] >= 0 && h >= 0 && h != g[r];
      const uint64_t ballot = __ballot(pair);
      if (ballot == 0) continue;  // uniform per wave
      int base = 0;
      if (lane == 0) base = atomicAdd(&n_list, int(__popcll(ballot)));
      base = __builtin_amdgcn_readfirstlane(base);
      const unsigned below = __builtin_amdgcn_mbcnt_hi(uint32_t(ballot >> 32),
                                                       __builtin_amdgcn_mbcnt_lo(uint32_t(ballot), 0u));
      if (pair) list[base + int(below)] = uint16_t(((yw + r) * kSlicTW + lane) * 2 + dir);
    }
  __syncthreads();
  const int n = n_list;
  for (int q = threadIdx.x; q < n; q += kDepthThreads) {
    const int code = list[q], dir = code & 1, px = code >> 1;
    const int64_t p = int64_t(y0 + px / kSlicTW) * K.W + x0 + px % kSlicTW;
    const int64_t o = dir == 0 ? p + 1 : p + K.W;
    double X[3], Y[3], C;
    load_xyz<DT>(arena, K.off + p, X, C);
    load_xyz<DT>(arena, K.off + o, Y, C);
    long long v = llrint((log_range(X) - log_range(Y)) * kFix);
    int gl = lab[p] - K.seg_base, hl = lab[o] - K.seg_base;
    if (gl > hl) {  // the pair at its lower segment, with that sign
      const int t = gl;
      gl = hl;
      hl = t;
      v = -v;
    }
    const int k = gl * kSlots + slot_of(K, gl, hl);
    int at = int(unsigned(k) * 2654435761u >> 23) & (kPairHash - 1), probe = 0;
    for (; probe < kPairProbes; ++probe, at = (at + 1) & (kPairHash - 1)) {
      const int was = atomicCAS(&key[at], -1, k);
      if (was == -1 || was == k) break;
    }
    if (probe < kPairProbes) {
      atomicAdd(&sum[at], (unsigned long long)v);
      atomicAdd(&cnt[at], 1);
    } else {
      add_pair(bsum, bcnt, K, gl, hl, (unsigned long long)v, 1);
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < kPairHash; q += kDepthThreads) {
    if (cnt[q] == 0) continue;
    const int gl = key[q] / kSlots, slot = key[q] - gl * kSlots;
    const int hl = gl + (slot / 7 - 3) * K.nx + (slot % 7 - 3);
    add_pair(bsum, bcnt, K, gl, hl, sum[q], cnt[q]);
  }
}

// ---- refinement iteration -------------------------------------------------------------------------------
struct DepthEdge {
  int64_t off_i, off_j, idx_off;
  int32_t npx_i, npx_j;
  int32_t base_i, base_j;  // first global segment id of keyframes i and j
  int32_t n_tiles;
  int32_t W_j;
};

// One block per (edge, tile of keyframe j): data-term sums of the segments it touches, flushed with float64
// atomics; the block's cost into its partial. The scale factors exp(eta) of both keyframes' segments are
// formed once per block into LDS. A block takes 64 x 64 pixels of j, a wave 64 columns by 16 rows, one row per step, so
// that every load, the gathers through the matches among them, covers few cache lines, and a lane goes down one column,
// where it stays in one segment of either keyframe for tens of rows (segments are that tall, and neighbouring matches
// land in neighbouring pixels of i): it sums in registers and adds to LDS when its segment changes. What the lanes hold
// at the end is summed over runs of 16 lanes first, since LDS adds to one address queue. 800 edges with 126.6 M pixels in
// bfloat16: 0.44 ms, 1.7 GB from memory (matches 4 B, points 8 B and slots 2 B at both ends, those of j shared); with four
// consecutive pixels per thread it took 0.70 ms, the address units busy 84% of it. Adding every match's sums through a
// segmented scan of a 64-pixel row held the same loads back to 0.60 ms (0.35 ms without the adds).
constexpr int kDataTile = 64;                                          // columns and rows per block
constexpr int kDataRows = kDataTile / (kDepthThreads / kWave);         // rows per wave
static_assert(kDataTile == kWave, "a lane per column");

// One step of the segmented inclusive scan over a row of 16 lanes: adds the sums of the lane D below unless a run starts
// in between (`head`, which then also covers that lane's reach).
template <int D>
__device__ inline void scan_step(int& head, float& h, float& g) {
  constexpr int kShr = 0x110 + D;  // row_shr:D; lanes below the row read 0 (a head there is set anyway)
  const float ph = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(h), kShr, 0xf, 0xf, true));
  const float pg = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(g), kShr, 0xf, 0xf, true));
  const int pf = __builtin_amdgcn_update_dpp(0, head, kShr, 0xf, 0xf, true);
  if (!head) {
    h += ph;
    g += pg;
  }
  head |= pf;
}

// The sums of 64 neighbouring columns by segment slot: runs of one slot within a row of 16 lanes are summed and their
// last lane adds them.
__device__ inline void merge_flush(float* H, float* G, uint32_t slot, float h, float g, int lane) {
  const uint32_t below = uint32_t(__builtin_amdgcn_update_dpp(0, int(slot), 0x111, 0xf, 0xf, true));  // row_shr:1
  int head = ((lane & 15) == 0 || below != slot) ? 1 : 0;
  const int next = __builtin_amdgcn_update_dpp(1, head, 0x101, 0xf, 0xf, false);  // row_shl:1, 1 past the row's end
  scan_step<1>(head, h, g);
  scan_step<2>(head, h, g);
  scan_step<4>(head, h, g);
  scan_step<8>(head, h, g);
  if (next && slot != kNoSlot) {
    atomicAdd(&H[slot], h);
    atomicAdd(&G[slot], g);
  }
}

template <int DT>
__global__ __launch_bounds__(kDepthThreads) void k_dr_data(const void* __restrict__ arena,
                                                           const DepthEdge* __restrict__ edges,
                                                           const int2* __restrict__ items,
                                                           const EdgeXf* __restrict__ xf,
                                                           const int32_t* __restrict__ idx_arena,
                                                           const uint16_t* __restrict__ slot,
                                                           const double* __restrict__ eta, int n_seg, DepthConst dc,
                                                           double* __restrict__ Hd, double* __restrict__ gd,
                                                           float* __restrict__ cost_part) {
  constexpr int kWaves = kDepthThreads / kWave;
  __shared__ float sHj[kMaxSegPerKf], sGj[kMaxSegPerKf], sHi[kMaxSegPerKf], sGi[kMaxSegPerKf];
  __shared__ float sEj[kMaxSegPerKf], sEi[kMaxSegPerKf];  // exp(eta) of the two keyframes' segments, eq. (8)
  __shared__ float red[kWaves];
  const int2 W = items[blockIdx.x];
  const DepthEdge E = edges[W.x];
  for (int q = threadIdx.x; q < kMaxSegPerKf; q += kDepthThreads) {
    sHj[q] = sGj[q] = sHi[q] = sGi[q] = 0.0f;
    sEj[q] = (E.base_j + q < n_seg) ? expf(float(eta[E.base_j + q])) : 1.0f;
    sEi[q] = (E.base_i + q < n_seg) ? expf(float(eta[E.base_i + q])) : 1.0f;
  }
  __syncthreads();
  float M[12];
#pragma unroll
  for (int q = 0; q < 12; ++q) M[q] = xf[W.x].m[q];
  const int32_t* __restrict__ idx = idx_arena + E.idx_off;
  float cost = 0.0f;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int tiles_x = (E.W_j + kDataTile - 1) / kDataTile;
  const int ty = W.y / tiles_x;
  const int x = (W.y - ty * tiles_x) * kDataTile + lane;
  const int y0 = ty * kDataTile + __builtin_amdgcn_readfirstlane(wave) * kDataRows;  // first row of the wave
  const int rows = min(kDataRows, E.npx_j / E.W_j - y0);
  struct Pt {
    typename Px<DT>::raw_t rj, ri;
    uint32_t h, g;
    int m;
  };
  auto load_match = [&](int k) {
    const int m = (k < rows && x < E.W_j) ? __builtin_nontemporal_load(idx + int64_t(y0 + k) * E.W_j + x) : -1;
    return m < E.npx_i ? m : -1;
  };
  // both points and slots of a match, without a branch (lanes without one read pixel 0)
  auto load_points = [&](int k, int m) {
    Pt P;
    const int64_t pj = E.off_j + (m >= 0 ? int64_t(y0 + k) * E.W_j + x : 0), pi = E.off_i + max(m, 0);
    P.m = m;
    P.rj = Px<DT>::load_raw(arena, pj);
    P.ri = Px<DT>::load_raw(arena, pi);
    P.h = slot[pj];
    P.g = slot[pi];
    return P;
  };
  uint32_t sj = kNoSlot, si = kNoSlot;  // the lane's open runs in j and in i, and their sums
  float hj = 0.0f, gj = 0.0f, hi = 0.0f, gi = 0.0f;
  // a pipeline over the rows: the points of the next row and the match words of the one after it are in flight while a
  // row is computed
  Pt cur = load_points(0, load_match(0));
  int ahead = load_match(1);
#pragma unroll 1
  for (int k = 0; k < rows; ++k) {
    const Pt P = cur;
    cur = load_points(k + 1, ahead);
    ahead = load_match(k + 2);
    if (__ballot(P.m >= 0) == 0) continue;  // uniform per wave
    const float4 A = Px<DT>::unpack(P.rj), B = Px<DT>::unpack(P.ri);
    const float dj2 = fmaf(A.x, A.x, fmaf(A.y, A.y, A.z * A.z));
    const float di2 = fmaf(B.x, B.x, fmaf(B.y, B.y, B.z * B.z));
    const float cc = B.w * A.w;
    const bool ok = P.m >= 0 && fminf(dj2, di2) > 1e-18f && dj2 + di2 + cc < __builtin_huge_valf() && cc >= 0.0f;
    const bool in_j = ok && P.h != kNoSlot, in_i = ok && P.g != kNoSlot;
    const float fh = in_j ? sEj[P.h] : 1.0f;  // exp(0) for a pixel without a segment
    const float fg = in_i ? sEi[P.g] : 1.0f;
    const float a0 = A.x * fh, a1 = A.y * fh, a2 = A.z * fh;  // X_j(eta), eq. (8)
    const float b0 = B.x * fg, b1 = B.y * fg, b2 = B.z * fg;  // X_i(eta)
    const float s = __builtin_amdgcn_sqrtf(__builtin_amdgcn_sqrtf(cc)) * dc.inv_sigma;
    const float R0 = fmaf(M[0], a0, fmaf(M[1], a1, M[2] * a2));  // sR_ij X_j(eta)
    const float R1 = fmaf(M[3], a0, fmaf(M[4], a1, M[5] * a2));
    const float R2 = fmaf(M[6], a0, fmaf(M[7], a1, M[8] * a2));
    const float r0 = s * (R0 + M[9] - b0), r1 = s * (R1 + M[10] - b1), r2 = s * (R2 + M[11] - b2);
    const float e0 = fabsf(r0), e1 = fabsf(r1), e2 = fabsf(r2);
    const float w0 = fminf(1.0f, dc.kappa * __builtin_amdgcn_rcpf(e0));
    const float w1 = fminf(1.0f, dc.kappa * __builtin_amdgcn_rcpf(e1));
    const float w2 = fminf(1.0f, dc.kappa * __builtin_amdgcn_rcpf(e2));
    const float t0 = w0 * e0, t1 = w1 * e1, t2 = w2 * e2;
    const float rho = t0 * fmaf(-0.5f, t0, e0) + t1 * fmaf(-0.5f, t1, e1) + t2 * fmaf(-0.5f, t2, e2);
    cost += ok ? rho : 0.0f;
    if (in_j && P.h != sj) {
      if (sj != kNoSlot) {
        atomicAdd(&sHj[sj], hj);
        atomicAdd(&sGj[sj], gj);
      }
      sj = P.h;
      hj = gj = 0.0f;
    }
    if (in_i && P.g != si) {
      if (si != kNoSlot) {
        atomicAdd(&sHi[si], hi);
        atomicAdd(&sGi[si], gi);
      }
      si = P.g;
      hi = gi = 0.0f;
    }
    const float J0 = s * R0, J1 = s * R1, J2 = s * R2;
    const float I0 = -s * b0, I1 = -s * b1, I2 = -s * b2;
    hj += in_j ? w0 * J0 * J0 + w1 * J1 * J1 + w2 * J2 * J2 : 0.0f;
    gj += in_j ? w0 * J0 * r0 + w1 * J1 * r1 + w2 * J2 * r2 : 0.0f;
    hi += in_i ? w0 * I0 * I0 + w1 * I1 * I1 + w2 * I2 * I2 : 0.0f;
    gi += in_i ? w0 * I0 * r0 + w1 * I1 * r1 + w2 * I2 * r2 : 0.0f;
  }
  merge_flush(sHj, sGj, sj, hj, gj, lane);
  merge_flush(sHi, sGi, si, hi, gi, lane);
  float c = wave_sum(cost);
  if (lane == 0) red[wave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.0f;
    for (int w = 0; w < kWaves; ++w) t += red[w];
    cost_part[blockIdx.x] = t;
  }
  for (int q = threadIdx.x; q < kMaxSegPerKf; q += kDepthThreads) {
    if (sHj[q] != 0.0f || sGj[q] != 0.0f) {
      atomicAdd(&Hd[E.base_j + q], double(sHj[q]));
      atomicAdd(&gd[E.base_j + q], double(sGj[q]));
    }
    if (sHi[q] != 0.0f || sGi[q] != 0.0f) {
      atomicAdd(&Hd[E.base_i + q], double(sHi[q]));
      atomicAdd(&gd[E.base_i + q], double(sGi[q]));
    }
  }
}

// kStepLanes lanes per segment, each on a few of its boundary slots (a thread per segment walks 49 slots of its own
// cache lines: 40 us for 43000 segments, 15 us this way): boundary and prior terms, the damped and clipped step (free
// segments only), and the segment's share of the boundary and prior cost (each unordered pair once, at its lower id).
// Each block also adds its share of the data kernel's cost partials and clears its segments' data sums for the next
// iteration.
constexpr int kStepLanes = 16;
constexpr int kStepSegs = kDepthThreads / kStepLanes;  // segments per block

__device__ inline double lanes16_sum(double v) {
#pragma unroll
  for (int off = kStepLanes / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

__global__ __launch_bounds__(kDepthThreads) void k_dr_step(const DepthKf* __restrict__ kfs, int n_kf,
                                                           const int32_t* __restrict__ seg_kf,
                                                           const uint8_t* __restrict__ seg_valid,
                                                           const unsigned long long* __restrict__ bsum,
                                                           const int32_t* __restrict__ bcnt,
                                                           double* __restrict__ Hd, double* __restrict__ gd,
                                                           const double* __restrict__ eta, double* __restrict__ eta_out,
                                                           int n_seg, DepthConst dc,
                                                           const float* __restrict__ data_part, int n_data,
                                                           double* __restrict__ cost_part) {
  const int s = blockIdx.x * kStepSegs + threadIdx.x / kStepLanes;
  const int lane = threadIdx.x % kStepLanes;
  double cost = 0.0;
  for (int q = blockIdx.x * kDepthThreads + threadIdx.x; q < n_data; q += gridDim.x * kDepthThreads)
    cost += double(data_part[q]);
  if (s < n_seg) {  // uniform per segment's lanes
    const double e = eta[s];
    double out = e;
    if (seg_valid[s]) {
      const DepthKf K = kfs[seg_kf[s]];
      const int l = s - K.seg_base;
      const int gy = l / K.nx, gx = l - gy * K.nx;
      double H = 0.0, g = 0.0;
      for (int q = lane; q < kSlots; q += kStepLanes) {
        const int c = bcnt[int64_t(s) * kSlots + q];
        if (c == 0) continue;
        const int hx = gx + q % 7 - 3, hy = gy + q / 7 - 3;
        const int h = K.seg_base + hy * K.nx + hx;
        const double dlt = double((long long)bsum[int64_t(s) * kSlots + q]) / kFix / double(c);
        const double rb = e - eta[h] + dlt;
        H += dc.lambda_smooth;
        g += dc.lambda_smooth * rb;
        if (s < h) cost += 0.5 * dc.lambda_smooth * rb * rb;
      }
      H = lanes16_sum(H) + (Hd[s] + dc.lambda_prior);
      g = lanes16_sum(g) + (gd[s] + dc.lambda_prior * e);
      if (lane == 0) cost += 0.5 * dc.lambda_prior * e * e;
      if (!K.anchor) {
        const double d = fmin(fmax(-g / ((1.0 + dc.lambda_lm) * H), -dc.eta_max), dc.eta_max);
        out = e + d;
      }
    }
    if (lane == 0) {
      eta_out[s] = out;
      Hd[s] = 0.0;
      gd[s] = 0.0;
    }
  }
  __shared__ double red[kDepthThreads / kWave];
  const double c = wave_sum(cost);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kDepthThreads / kWave; ++w) t += red[w];
    cost_part[blockIdx.x] = t;
  }
}

// Cost of the iteration: the step kernel's partials summed in a fixed order into hist[it].
__global__ __launch_bounds__(kDepthThreads) void k_dr_cost(const double* __restrict__ step_part, int n_step,
                                                           double* __restrict__ hist, int it) {
  double acc = 0.0;
  for (int q = threadIdx.x; q < n_step; q += kDepthThreads) acc += step_part[q];
  __shared__ double red[kDepthThreads / kWave];
  const double c = wave_sum(acc);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kDepthThreads / kWave; ++w) t += red[w];
    hist[it] = t;
  }
}

// Plan facts: valid segments into facts[0], boundary slots in use into facts[1] (both cleared before). One small copy to
// the host instead of the whole table (8.4 MB and a walk over 2.1 M counts for 43000 segments).
__global__ __launch_bounds__(kDepthThreads) void k_dr_facts(const uint8_t* __restrict__ seg_valid, int n_seg,
                                                            const int32_t* __restrict__ bcnt,
                                                            unsigned long long* __restrict__ facts) {
  const int64_t stride = int64_t(gridDim.x) * kDepthThreads, n = int64_t(n_seg) * kSlots;
  int v = 0, p = 0;
  for (int64_t q = int64_t(blockIdx.x) * kDepthThreads + threadIdx.x; q < n; q += stride) {
    if (q < n_seg) v += seg_valid[q];
    p += bcnt[q] > 0;
  }
  v = wave_sum(v);
  p = wave_sum(p);
  if ((threadIdx.x & (kWave - 1)) == 0) {
    if (v) atomicAdd(&facts[0], (unsigned long long)v);
    if (p) atomicAdd(&facts[1], (unsigned long long)p);
  }
}

// X(eta) for every arena pixel: xyz scaled by exp(eta_g), confidence copied (float32 xyzc out).
template <int DT>
__global__ __launch_bounds__(kDepthThreads) void k_dr_apply(const void* __restrict__ arena, int64_t n_px,
                                                            const int32_t* __restrict__ label,
                                                            const double* __restrict__ eta, float4* __restrict__ out) {
  const int64_t p = int64_t(blockIdx.x) * kDepthThreads + threadIdx.x;
  if (p >= n_px) return;
  const float4 X = Px<DT>::load(arena, p);
  const int g = label[p];
  const double f = g >= 0 ? exp(eta[g]) : 1.0;
  out[p] = make_float4(float(double(X.x) * f), float(double(X.y) * f), float(double(X.z) * f), X.w);
}

// ---- plan -----------------------------------------------------------------------------------------------
struct DepthPlan {
  ds3_dtype dt = DS3_F32;
  const void* arena = nullptr;
  const int32_t* idx = nullptr;
  int n_kf = 0, n_edges = 0, n_seg = 0, n_items = 0;
  int64_t n_px = 0;
  DepthConst dc;
  std::vector<DepthKf> kf_host;
  void* mem = nullptr;
  DepthKf* kfs = nullptr;
  DepthEdge* edges = nullptr;
  EdgeDev* gedges = nullptr;  // for the pose prep
  int2* items = nullptr;
  EdgeXf* xf = nullptr;
  double* Ad = nullptr;
  int32_t* label = nullptr;
  uint2* feat = nullptr;
  uint16_t* slot = nullptr;  // per pixel: segment slot of its keyframe; shares feat's memory once the labels are final
  int64_t* cen = nullptr;
  unsigned long long* sums = nullptr;  // per segment: members, then the sums of x, y and the four features
  int32_t* cnt = nullptr;
  uint8_t* seg_valid = nullptr;
  int32_t* seg_kf = nullptr;
  unsigned long long* bsum = nullptr;
  int32_t* bcnt = nullptr;
  double *eta = nullptr, *eta2 = nullptr, *Hd = nullptr, *gd = nullptr;
  double *lmin = nullptr, *lmax = nullptr, *range = nullptr;
  float* data_part = nullptr;
  double* step_part = nullptr;
  double* hist = nullptr;
  int64_t valid_segments = 0, pairs = 0, px_scanned = 0;
};

static size_t carve_depth(void* base, DepthPlan& P) {
  Carver c(base);
  P.kfs = c.take<DepthKf>(P.n_kf);
  P.edges = c.take<DepthEdge>(std::max(P.n_edges, 1));
  P.gedges = c.take<EdgeDev>(std::max(P.n_edges, 1));
  P.items = c.take<int2>(std::max(P.n_items, 1));
  P.xf = c.take<EdgeXf>(std::max(P.n_edges, 1));
  P.Ad = c.take<double>(49 * size_t(std::max(P.n_edges, 1)));
  P.label = c.take<int32_t>(size_t(P.n_px));
  P.feat = c.take<uint2>(size_t(P.n_px));
  P.slot = reinterpret_cast<uint16_t*>(P.feat);
  P.cen = c.take<int64_t>(6 * size_t(P.n_seg));
  P.sums = c.take<unsigned long long>(7 * size_t(P.n_seg));
  P.cnt = c.take<int32_t>(P.n_seg);
  P.seg_valid = c.take<uint8_t>(P.n_seg);
  P.seg_kf = c.take<int32_t>(P.n_seg);
  P.bsum = c.take<unsigned long long>(size_t(kSlots) * P.n_seg);
  P.bcnt = c.take<int32_t>(size_t(kSlots) * P.n_seg);
  P.eta = c.take<double>(P.n_seg);
  P.eta2 = c.take<double>(P.n_seg);
  P.Hd = c.take<double>(P.n_seg);
  P.gd = c.take<double>(P.n_seg);
  P.lmin = c.take<double>(size_t(P.n_kf) * kRangeParts);
  P.lmax = c.take<double>(size_t(P.n_kf) * kRangeParts);
  P.range = c.take<double>(3 * size_t(P.n_kf));
  P.data_part = c.take<float>(std::max(P.n_items, 1));
  P.step_part = c.take<double>((P.n_seg + kStepSegs - 1) / kStepSegs);
  P.hist = c.take<double>(1024);
  return c.used;
}

template <class T>
static int upload_vec(T* dst, const std::vector<T>& src, hipStream_t s) {
  if (src.empty()) return DS3_OK;
  return check_hip(hipMemcpyAsync(dst, src.data(), sizeof(T) * src.size(), hipMemcpyHostToDevice, s), "upload");
}

static void launch_range(DepthPlan& P, hipStream_t s) {
  hipLaunchKernelGGL(k_dr_range, dim3((P.n_kf + 63) / 64), dim3(64), 0, s, P.n_kf, P.lmin, P.lmax, P.range);
}

static int depth_segment(DepthPlan& P, int slic_iters, int min_px, hipStream_t s) {
  int max_px = 0, max_m = 0, max_side = 0;
  int64_t max_tiles = 0;
  for (auto& K : P.kf_host) {
    max_px = std::max(max_px, K.H * K.W);
    max_m = std::max(max_m, K.nx * K.ny);
    max_side = std::max(max_side, std::max(K.H, K.W));
    max_tiles = std::max(max_tiles, int64_t((K.W + kSlicTW - 1) / kSlicTW) * ((K.H + kSlicTH - 1) / kSlicTH));
  }
  const dim3 gpass(unsigned(max_tiles), P.n_kf), grange(kRangeParts, P.n_kf);
  const dim3 gpx((max_px + kDepthThreads - 1) / kDepthThreads, P.n_kf);
  if (P.dt == DS3_F32) {
    hipLaunchKernelGGL(k_dr_logrange<DS3_F32>, grange, dim3(kDepthThreads), 0, s, P.arena, P.kfs, P.dc, P.lmin, P.lmax);
    launch_range(P, s);
    hipLaunchKernelGGL(k_dr_features<DS3_F32>, gpx, dim3(kDepthThreads), 0, s, P.arena, P.kfs, P.dc, P.range, P.feat);
  } else {
    hipLaunchKernelGGL(k_dr_logrange<DS3_BF16>, grange, dim3(kDepthThreads), 0, s, P.arena, P.kfs, P.dc, P.lmin, P.lmax);
    launch_range(P, s);
    hipLaunchKernelGGL(k_dr_features<DS3_BF16>, gpx, dim3(kDepthThreads), 0, s, P.arena, P.kfs, P.dc, P.range, P.feat);
  }
  DS3_TRY(check_hip(hipGetLastError(), "k_dr_features"));
  hipLaunchKernelGGL(k_slic_init, dim3((max_m + 63) / 64, P.n_kf), dim3(64), 0, s, P.kfs, P.n_kf, P.feat, P.cen);
  DS3_TRY(check_hip(hipGetLastError(), "k_slic_init"));
  DS3_TRY(launch_fill_u32(reinterpret_cast<unsigned*>(P.sums), 14 * size_t(P.n_seg), 0u, s));
  for (int it = 0; it < slic_iters; ++it) {
    const int last = it == slic_iters - 1;
    if (max_side > 32767)
      hipLaunchKernelGGL(k_slic_pass<true>, gpass, dim3(kDepthThreads), 0, s, P.kfs, P.feat, P.cen, P.sums, P.label, last);
    else
      hipLaunchKernelGGL(k_slic_pass<false>, gpass, dim3(kDepthThreads), 0, s, P.kfs, P.feat, P.cen, P.sums, P.label, last);
    hipLaunchKernelGGL(k_slic_move, dim3((P.n_seg + kDepthThreads - 1) / kDepthThreads), dim3(kDepthThreads), 0, s,
                       P.sums, P.n_seg, P.cen, P.cnt);
    DS3_TRY(check_hip(hipGetLastError(), "k_slic"));
  }
  const dim3 gfin((std::max(max_px, max_m) + kDepthThreads - 1) / kDepthThreads, P.n_kf);
  hipLaunchKernelGGL(k_label_finalize, gfin, dim3(kDepthThreads), 0, s, P.kfs, P.cnt, min_px, P.label, P.slot, P.seg_valid);
  DS3_TRY(check_hip(hipGetLastError(), "k_label_finalize"));
  DS3_TRY(launch_fill_u32(reinterpret_cast<unsigned*>(P.bsum), 2 * kSlots * size_t(P.n_seg), 0u, s));
  DS3_TRY(launch_fill_u32(reinterpret_cast<unsigned*>(P.bcnt), kSlots * size_t(P.n_seg), 0u, s));
  if (P.dt == DS3_F32)
    hipLaunchKernelGGL(k_dr_boundary<DS3_F32>, gpass, dim3(kDepthThreads), 0, s, P.arena, P.kfs, P.label, P.bsum, P.bcnt);
  else
    hipLaunchKernelGGL(k_dr_boundary<DS3_BF16>, gpass, dim3(kDepthThreads), 0, s, P.arena, P.kfs, P.label, P.bsum, P.bcnt);
  return check_hip(hipGetLastError(), "k_dr_boundary");
}

// The data term's blocks (edge, tile). Block b runs on XCD b mod 8: each XCD takes a run of the list that has the edges of
// one tile of a keyframe j side by side, so that they share its points and slots in that XCD's L2 (1.67 GB from memory
// instead of 2.48 GB, 438 us instead of 453 us, for 800 edges of 200 keyframes).
static std::vector<int2> data_items(const std::vector<DepthEdge>& edges, int n_edges) {
  std::vector<int> by_j(n_edges);
  for (int e = 0; e < n_edges; ++e) by_j[e] = e;
  std::stable_sort(by_j.begin(), by_j.end(), [&](int a, int b) { return edges[a].off_j < edges[b].off_j; });
  size_t n = 0;
  for (int e = 0; e < n_edges; ++e) n += size_t(edges[e].n_tiles);
  std::vector<int2> out(n);
  // item p of the list, in its XCD's run, goes to block 8 (p - run's first) + XCD; the first n % 8 runs have one more
  const size_t per = n / 8, extra = n % 8;
  size_t xcd = 0, at = 0;
  auto put = [&](int e, int t) {
    while (at == per + (xcd < extra ? 1 : 0)) {
      ++xcd;
      at = 0;
    }
    out[8 * at + xcd] = make_int2(e, t);
    ++at;
  };
  for (int first = 0, last; first < n_edges; first = last) {
    int tiles = 0;
    for (last = first; last < n_edges && edges[by_j[last]].off_j == edges[by_j[first]].off_j; ++last)
      tiles = std::max(tiles, edges[by_j[last]].n_tiles);
    for (int t = 0; t < tiles; ++t)
      for (int k = first; k < last; ++k)
        if (t < edges[by_j[k]].n_tiles) put(by_j[k], t);
  }
  return out;
}

static void depth_free(DepthPlan* P) {
  if (!P) return;
  if (P->mem) (void)hipFree(P->mem);
  delete P;
}

}  // namespace ds3

using namespace ds3;

extern "C" {

void ds3_default_depth_params(ds3_depth_params* p) {
  if (!p) return;
  p->segments_per_kf = 200;
  p->conf_min = 1.5;
  p->min_seg_px = 16;
  p->slic_iters = 10;
  p->sigma_point = 0.05;
  p->huber_k = 1.345;
  p->lambda_smooth = 1.0;
  p->lambda_prior = 1.0;
  p->lambda_lm = 0.05;
  p->eta_max = 0.5;
}

int ds3_depth_plan_create(int32_t n_kf, const ds3_image* kf, const void* arena, ds3_dtype dtype, const ds3_edge* edges,
                          int32_t n_edges, const int32_t* idx_arena, const int32_t* anchors, int32_t n_anchors,
                          const ds3_depth_params* params, void** plan_out, void* stream) {
  if (!plan_out) return fail(DS3_EINVAL, "depth: plan_out is null");
  *plan_out = nullptr;
  if (n_kf <= 0 || !kf || !arena || !params || n_edges < 0 || (n_edges > 0 && (!edges || !idx_arena)) ||
      n_anchors < 0 || (n_anchors > 0 && !anchors))
    return fail(DS3_EINVAL, "depth: bad arguments");
  if (dtype != DS3_F32 && dtype != DS3_BF16) return fail(DS3_ENOTSUP, "depth: dtype");
  if ((reinterpret_cast<uintptr_t>(arena) & 15) != 0) return fail(DS3_EINVAL, "depth: arena must be 16 B aligned");
  const ds3_depth_params& p = *params;
  if (p.segments_per_kf < 1 || p.min_seg_px < 0 || p.slic_iters < 1 || p.slic_iters > 100 || !(p.sigma_point > 0) ||
      !(p.huber_k > 0) || !(p.lambda_smooth >= 0) || !(p.lambda_prior >= 0) || !(p.lambda_lm >= 0) ||
      !(p.eta_max > 0))
    return fail(DS3_EINVAL, "depth: bad parameters");
  DepthPlan* P = new DepthPlan();
  P->dt = dtype;
  P->arena = arena;
  P->idx = idx_arena;
  P->n_kf = n_kf;
  P->n_edges = n_edges;
  P->dc.conf_min = p.conf_min;
  P->dc.inv_sigma = float(1.0 / p.sigma_point);
  P->dc.kappa = float(p.huber_k);
  P->dc.lambda_smooth = p.lambda_smooth;
  P->dc.lambda_prior = p.lambda_prior;
  P->dc.lambda_lm = p.lambda_lm;
  P->dc.eta_max = p.eta_max;
  std::vector<uint8_t> is_anchor(n_kf, 0);
  for (int a = 0; a < n_anchors; ++a) {
    if (anchors[a] < 0 || anchors[a] >= n_kf) { depth_free(P); return fail(DS3_EINVAL, "depth: anchor out of range"); }
    is_anchor[anchors[a]] = 1;
  }
  int seg = 0;
  int64_t px = 0;
  std::vector<int32_t> seg_kf;
  for (int k = 0; k < n_kf; ++k) {
    const ds3_image& I = kf[k];
    if (I.H <= 0 || I.W <= 0 || I.px_offset < 0 || int64_t(I.H) * I.W > INT32_MAX) {
      depth_free(P);
      return fail(DS3_EINVAL, "depth: bad keyframe image " + std::to_string(k));
    }
    DepthKf K;
    K.off = I.px_offset;
    K.H = I.H;
    K.W = I.W;
    K.S = std::max(1, int(std::floor(std::sqrt(double(I.H) * I.W / p.segments_per_kf) + 0.5)));
    K.nx = (I.W + K.S - 1) / K.S;
    K.ny = (I.H + K.S - 1) / K.S;
    if (K.nx * K.ny > kMaxSegPerKf) {
      depth_free(P);
      return fail(DS3_EINVAL, "depth: more than 256 segments in keyframe " + std::to_string(k));
    }
    K.seg_base = seg;
    K.anchor = is_anchor[k];
    K.pad = 0;
    for (int q = 0; q < K.nx * K.ny; ++q) seg_kf.push_back(k);
    seg += K.nx * K.ny;
    px = std::max(px, I.px_offset + int64_t(I.H) * I.W);
    P->kf_host.push_back(K);
  }
  P->n_seg = seg;
  P->n_px = px;
  // edges and their tiles
  std::vector<DepthEdge> de(std::max(n_edges, 1));
  std::vector<EdgeDev> ge(std::max(n_edges, 1));
  for (int e = 0; e < n_edges; ++e) {
    const ds3_edge& Ed = edges[e];
    if (Ed.i < 0 || Ed.i >= n_kf || Ed.j < 0 || Ed.j >= n_kf || Ed.i == Ed.j || Ed.idx_offset < 0) {
      depth_free(P);
      return fail(DS3_EINVAL, "depth: bad edge " + std::to_string(e));
    }
    DepthEdge D;
    D.off_i = kf[Ed.i].px_offset;
    D.off_j = kf[Ed.j].px_offset;
    D.idx_off = Ed.idx_offset;
    D.npx_i = kf[Ed.i].H * kf[Ed.i].W;
    D.npx_j = kf[Ed.j].H * kf[Ed.j].W;
    D.base_i = P->kf_host[Ed.i].seg_base;
    D.base_j = P->kf_host[Ed.j].seg_base;
    D.W_j = kf[Ed.j].W;
    const int64_t n_tiles = int64_t((kf[Ed.j].W + kDataTile - 1) / kDataTile) * ((kf[Ed.j].H + kDataTile - 1) / kDataTile);
    D.n_tiles = int32_t(n_tiles);
    de[e] = D;
    EdgeDev G{};
    G.off_i = D.off_i;
    G.off_j = D.off_j;
    G.idx_off = D.idx_off;
    G.npx_i = D.npx_i;
    G.npx_j = D.npx_j;
    G.i = Ed.i;
    G.j = Ed.j;
    ge[e] = G;
    P->px_scanned += D.npx_j;
  }
  const std::vector<int2> items = data_items(de, n_edges);
  P->n_items = int(items.size());
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t bytes = carve_depth(nullptr, *P);
  int rc = check_hip(hipMalloc(&P->mem, bytes), "hipMalloc(depth plan)");
  if (rc == DS3_OK) {
    carve_depth(P->mem, *P);
    rc = upload_vec(P->kfs, P->kf_host, s);
    if (rc == DS3_OK) rc = upload_vec(P->edges, de, s);
    if (rc == DS3_OK) rc = upload_vec(P->gedges, ge, s);
    if (rc == DS3_OK) rc = upload_vec(P->items, items, s);
    if (rc == DS3_OK) rc = upload_vec(P->seg_kf, seg_kf, s);
    if (rc == DS3_OK) rc = launch_fill(P->eta, size_t(P->n_seg), 0.0, s);
    if (rc == DS3_OK) rc = launch_fill(P->Hd, size_t(P->n_seg), 0.0, s);
    if (rc == DS3_OK) rc = launch_fill(P->gd, size_t(P->n_seg), 0.0, s);
    if (rc == DS3_OK) rc = depth_segment(*P, p.slic_iters, p.min_seg_px, s);
    // facts for the caller (synchronises once, at creation)
    unsigned long long facts[2] = {0, 0};
    unsigned long long* d_facts = reinterpret_cast<unsigned long long*>(P->hist);  // written by runs only
    if (rc == DS3_OK) rc = launch_fill_u32(reinterpret_cast<unsigned*>(d_facts), 4, 0u, s);
    if (rc == DS3_OK) {
      const int64_t blocks = (int64_t(P->n_seg) * kSlots + kDepthThreads - 1) / kDepthThreads;
      hipLaunchKernelGGL(k_dr_facts, dim3(unsigned(std::min<int64_t>(blocks, 256))), dim3(kDepthThreads), 0, s,
                         P->seg_valid, P->n_seg, P->bcnt, d_facts);
      rc = check_hip(hipGetLastError(), "k_dr_facts");
    }
    if (rc == DS3_OK) rc = check_hip(hipMemcpyAsync(facts, d_facts, sizeof(facts), hipMemcpyDeviceToHost, s), "d2h");
    if (rc == DS3_OK) rc = check_hip(hipStreamSynchronize(s), "hipStreamSynchronize(depth plan)");
    P->valid_segments = int64_t(facts[0]);
    P->pairs = int64_t(facts[1]);
  }
  if (rc != DS3_OK) { depth_free(P); return rc; }
  *plan_out = P;
  return DS3_OK;
}

int ds3_depth_plan_run(void* plan, const double* poses, int32_t iters, double* cost_per_iter, ds3_timer* data_timer,
                       void* stream) {
  DepthPlan* P = static_cast<DepthPlan*>(plan);
  if (!P || !poses || iters < 0 || iters > 1024) return fail(DS3_EINVAL, "depth_run: bad arguments");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nstep = (P->n_seg + kStepSegs - 1) / kStepSegs;
  if (iters > 0) DS3_TRY(launch_gn_prep(poses, P->gedges, P->n_edges, P->xf, P->Ad, s));  // the poses stay fixed
  for (int it = 0; it < iters; ++it) {
    const bool timed = data_timer && it == iters - 1;
    if (timed) DS3_TRY(timer_record(data_timer, true, s));
    if (P->n_items > 0) {
      if (P->dt == DS3_F32)
        hipLaunchKernelGGL(k_dr_data<DS3_F32>, dim3(P->n_items), dim3(kDepthThreads), 0, s, P->arena, P->edges, P->items,
                           P->xf, P->idx, P->slot, P->eta, P->n_seg, P->dc, P->Hd, P->gd, P->data_part);
      else
        hipLaunchKernelGGL(k_dr_data<DS3_BF16>, dim3(P->n_items), dim3(kDepthThreads), 0, s, P->arena, P->edges, P->items,
                           P->xf, P->idx, P->slot, P->eta, P->n_seg, P->dc, P->Hd, P->gd, P->data_part);
      DS3_TRY(check_hip(hipGetLastError(), "k_dr_data"));
    }
    if (timed) DS3_TRY(timer_record(data_timer, false, s));
    hipLaunchKernelGGL(k_dr_step, dim3(std::max(nstep, 1)), dim3(kDepthThreads), 0, s, P->kfs, P->n_kf, P->seg_kf,
                       P->seg_valid, P->bsum, P->bcnt, P->Hd, P->gd, P->eta, P->eta2, P->n_seg, P->dc, P->data_part,
                       P->n_items, P->step_part);
    DS3_TRY(check_hip(hipGetLastError(), "k_dr_step"));
    hipLaunchKernelGGL(k_dr_cost, dim3(1), dim3(kDepthThreads), 0, s, P->step_part, nstep, P->hist, it);
    DS3_TRY(check_hip(hipGetLastError(), "k_dr_cost"));
    std::swap(P->eta, P->eta2);
  }
  if (iters > 0 && cost_per_iter)
    DS3_TRY(check_hip(hipMemcpyAsync(cost_per_iter, P->hist, sizeof(double) * iters, hipMemcpyDeviceToDevice, s), "copy"));
  return DS3_OK;
}

int ds3_depth_plan_info(void* plan, int64_t* info, int32_t n_info) {
  DepthPlan* P = static_cast<DepthPlan*>(plan);
  if (!P || !info || n_info < 0) return fail(DS3_EINVAL, "depth_info: bad arguments");
  const int64_t v[6] = {P->n_seg, P->valid_segments, P->pairs, P->n_items, P->px_scanned, P->n_px};
  for (int k = 0; k < n_info && k < 6; ++k) info[k] = v[k];
  return DS3_OK;
}

int ds3_depth_plan_get(void* plan, int32_t* labels_out, double* eta_out, void* stream) {
  DepthPlan* P = static_cast<DepthPlan*>(plan);
  if (!P) return fail(DS3_EINVAL, "depth_get: null plan");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (labels_out)
    DS3_TRY(check_hip(hipMemcpyAsync(labels_out, P->label, sizeof(int32_t) * size_t(P->n_px), hipMemcpyDeviceToDevice, s),
                      "copy labels"));
  if (eta_out)
    DS3_TRY(check_hip(hipMemcpyAsync(eta_out, P->eta, sizeof(double) * size_t(P->n_seg), hipMemcpyDeviceToDevice, s),
                      "copy eta"));
  return DS3_OK;
}

int ds3_depth_plan_set_eta(void* plan, const double* eta, void* stream) {
  DepthPlan* P = static_cast<DepthPlan*>(plan);
  if (!P || !eta) return fail(DS3_EINVAL, "depth_set_eta: bad arguments");
  return check_hip(hipMemcpyAsync(P->eta, eta, sizeof(double) * size_t(P->n_seg), hipMemcpyDeviceToDevice,
                                  static_cast<hipStream_t>(stream)),
                   "copy eta");
}

int ds3_depth_plan_apply(void* plan, float* xyzc_out, void* stream) {
  DepthPlan* P = static_cast<DepthPlan*>(plan);
  if (!P || !xyzc_out) return fail(DS3_EINVAL, "depth_apply: bad arguments");
  if ((reinterpret_cast<uintptr_t>(xyzc_out) & 15) != 0) return fail(DS3_EINVAL, "depth_apply: output not 16 B aligned");
  if (P->n_px == 0) return DS3_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const dim3 g(unsigned((P->n_px + kDepthThreads - 1) / kDepthThreads));
  if (P->dt == DS3_F32)
    hipLaunchKernelGGL(k_dr_apply<DS3_F32>, g, dim3(kDepthThreads), 0, s, P->arena, P->n_px, P->label, P->eta,
                       reinterpret_cast<float4*>(xyzc_out));
  else
    hipLaunchKernelGGL(k_dr_apply<DS3_BF16>, g, dim3(kDepthThreads), 0, s, P->arena, P->n_px, P->label, P->eta,
                       reinterpret_cast<float4*>(xyzc_out));
  return check_hip(hipGetLastError(), "k_dr_apply");
}

int ds3_depth_plan_destroy(void* plan) {
  depth_free(static_cast<DepthPlan*>(plan));
  return DS3_OK;
}

}  // extern "C"
